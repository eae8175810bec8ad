"""Puts, page copies and row writes at the sizes where their launches split:
row counts around the two kernel-argument sizes, rows in more views than one
launch lists, value tensors that are not 16-byte aligned, every layer.
Gathers are compared bit for bit with the host's copy."""
import numpy as np
import pytest
import torch

from paper_2602_01519_amd import pic, runner
from paper_2602_01519_amd import workloads as W

from test_gpu_blend import stream

pytestmark = pytest.mark.gpu

LAYERS = 3


def bits(rng, shape, dtype):
    if dtype == W.BF16:
        return rng.integers(0, 1 << 16, shape, dtype=np.uint16)
    return rng.integers(0, 1 << 32, shape, dtype=np.uint32).view(np.float32)


def gathered(store, cid, n, kind, dtype, heads, d_k, d_v, layer):
    et = torch.float32 if dtype == W.F32 else torch.int16
    k = torch.empty((n, heads, d_k), dtype=et, device="cuda")
    v = None if kind == W.MLA else torch.empty((n, heads, d_v), dtype=et, device="cuda")
    pic.debug_gather(store, [cid], k, v, stream=stream(), layer=layer)
    torch.cuda.synchronize()
    return k.cpu().numpy().tobytes(), None if v is None else v.cpu().numpy().tobytes()


def offset_tensor(a, elements):
    """The host array on the device, its first element `elements` past a 16-byte boundary."""
    t = runner.to_device(a, "cuda")
    buf = torch.empty(t.numel() + elements, dtype=t.dtype, device="cuda")
    buf[elements:] = t.reshape(-1)
    return buf[elements:]


@pytest.mark.parametrize("kind,dtype,heads,d_k,d_v,n_rows", [
    (W.GQA, W.BF16, 3, 128, 128, 128), (W.GQA, W.BF16, 2, 64, 40, 129),
    (W.GQA, W.F32, 3, 24, 64, 768), (W.GQA, W.F32, 2, 64, 72, 769), (W.MLA, W.BF16, 1, 576, 512, 1),
    (W.GQA, W.BF16, 1, 8, 8, 1000)])
def test_rows_and_pages_bit_exact(kind, dtype, heads, d_k, d_v, n_rows):
    rng = np.random.default_rng(n_rows)
    n = 64 * 40 + 17
    store = pic.Store(kind, dtype, heads, d_k, d_v, 64 * 140, n_layers=LAYERS)
    try:
        # holes of one page, so that the derived chunk's private pages lie in many runs
        fill_k = bits(rng, (LAYERS, 64, heads, d_k), dtype)
        fill_v = None if kind == W.MLA else bits(rng, (LAYERS, 64, heads, d_v), dtype)
        for i in range(90):
            store.put(5000 + i, 64, runner.to_device(fill_k, "cuda"),
                      runner.to_device(fill_v, "cuda"), stream())
        k = bits(rng, (LAYERS, n, heads, d_k), dtype)
        v = None if kind == W.MLA else bits(rng, (LAYERS, n, heads, d_v), dtype)
        store.put(1, n, runner.to_device(k, "cuda"),
                  None if v is None else offset_tensor(v, 1), stream())
        for i in range(0, 90, 2):
            store.remove(5000 + i, stream())
        torch.cuda.synchronize()
        for l in range(LAYERS):
            gk, gv = gathered(store, 1, n, kind, dtype, heads, d_k, d_v, l)
            assert gk == k[l].tobytes() and (v is None or gv == v[l].tobytes()), f"put layer {l}"
        rows = np.sort(rng.choice(n, n_rows, replace=False)).astype(np.int32)
        store.derive(2, 1, rows, stream())
        for l in (2, 0, 1):
            nk = bits(rng, (n_rows, heads, d_k), dtype)
            nv = None if kind == W.MLA else bits(rng, (n_rows, heads, d_v), dtype)
            store.write_rows(2, l, rows, runner.to_device(nk, "cuda"),
                             None if nv is None else offset_tensor(nv, 3), stream())
            want_k, want_v = k[l].copy(), None if v is None else v[l].copy()
            want_k[rows] = nk
            if v is not None:
                want_v[rows] = nv
            gk, gv = gathered(store, 2, n, kind, dtype, heads, d_k, d_v, l)
            assert gk == want_k.tobytes() and (v is None or gv == want_v.tobytes()), f"layer {l}"
            gk, gv = gathered(store, 1, n, kind, dtype, heads, d_k, d_v, l)
            assert gk == k[l].tobytes(), f"base layer {l}"
    finally:
        store.close()
