"""The streaming matrix-core kernel for fp32 and narrow bf16 GQA calls at the
sizes where its tiling can go wrong: rows around a wave's 16 / 32 / 64 and a
workgroup's key parts, 32-key tiles that end inside a page, causal limits
inside a tile, link tables past 64 entries, its two call forms (tables in
device memory, tables as a kernel argument), against the fp64 oracle.

The probabilities of this kernel are fp32 (for bf16 caches the value product
takes them as a sum of two bf16 numbers, relative error <= 2^-17), so beyond
the bf16 parity bar its log-sum-exp has the fp32 bar and its output only the
rounding to bf16: |out - ref| <= 2^-8 |ref| + 2^-16 max|v| per element
(rounding to 8 significant bits; twice the split's 2^-17 bounds numerator
and denominator).
"""
import numpy as np
import pytest

import oracle
import parity_gate as G
from paper_2602_01519_amd import pic, runner
from paper_2602_01519_amd import workloads as W

from test_gpu_blend import ref_link, run_link, stream as cur_stream
from test_gpu_link import run_and_check

pytestmark = pytest.mark.gpu

# (dtype, d, query heads, kv heads, q_len, own beyond the query, chunk lengths, links, decode)
FORMS = {
    "one_row": (W.F32, 64, 3, 3, (1,) * 9, (0, 40, 31) * 3, (1, 31, 33), (1, 3), False),
    "rows_16_17": (W.F32, 32, 3, 1, (5, 6), (3, 0), (64, 65, 95), (2, 3), False),
    "rows_33_parts": (W.BF16, 64, 3, 1, (11, 12), (30, 33), (100, 700, 31), (2, 3), False),
    "rows_65_130": (W.BF16, 32, 5, 1, (13, 26), (0, 7), (96, 97, 640), (2, 3), False),
    "rows_129_own": (W.BF16, 64, 6, 2, (43, 44), (70, 0), (300, 33, 64), (1, 3), False),
    "f32_d128": (W.F32, 128, 6, 2, (43, 9), (0, 31), (300, 33, 64), (1, 3), False),
    "many_links": (W.BF16, 64, 6, 2, (9, 70), (5, 5), tuple(range(1, 80)), (66, 79), False),
    "decode": (W.BF16, 64, 24, 8, (1, 2), (70, 31), (700, 64, 333), (2, 3), True),
    "decode_f32": (W.F32, 32, 10, 2, (1, 3), (0, 64), (700, 64, 333), (2, 3), True),
    "nine_requests": (W.F32, 64, 6, 2, (1, 3, 2, 17, 40, 6, 5, 4, 31), (0,) * 9, (90, 200, 31),
                      (0, 3), False),
}


@pytest.mark.parametrize("name", sorted(FORMS))
def test_stream_forms(name):
    dtype, d, hq, hkv, q, extra, lens, links, decode = FORMS[name]
    cfg = W.small_config("stream_" + name, dtype=dtype, d_k=d, n_q_heads=hq, n_kv_heads=hkv,
                         chunk_lens=lens, batch=len(q), links=links, q_len=q,
                         self_len=tuple(a + b for a, b in zip(q, extra)), decode=decode)
    pic.prof_begin()
    try:
        out, lse = run_and_check(cfg)
    finally:
        _, _, ran = pic.prof_end()
    assert "stream" in ran, ran
    if dtype == W.BF16:
        wl = W.make_workload(cfg)
        chunks = {c: W.make_chunk(cfg, int(c)) for c in wl.used_chunks()}
        ref, ref_lse = oracle.run_workload(wl, chunks)
        fin = np.isfinite(ref_lse)
        assert np.abs(lse[fin] - ref_lse[fin]).max() <= G.TOL[G.F32].lse
        vmax = max([float(np.abs(W.bf16_bits_to_f32(v)).max()) for _, v in chunks.values()] +
                   [float(np.abs(W.bf16_bits_to_f32(wl.v_self)).max())])
        assert np.all(np.abs(out - ref) <= 2.0 ** -8 * np.abs(ref) + 2.0 ** -16 * vmax)


@pytest.mark.parametrize("dtype,d", [(W.F32, 64), (W.BF16, 64), (W.BF16, 32)])
def test_stream_limits(dtype, d):
    """Per-query limits on the linked rows inside, on and past tile edges."""
    cfg = W.small_config("stream_limits", dtype=dtype, d_k=d, n_q_heads=6, n_kv_heads=2,
                         chunk_lens=(70, 33, 130), batch=1, links=(3, 3), q_len=40,
                         self_len=None)
    wl = W.make_workload(cfg)
    p = wl.plan
    dw = runner.upload(wl)
    try:
        total = sum(cfg.chunk_length(int(c)) for c in p.chunk_index)
        edges = [0, 1, 31, 32, 33, 63, 64, 70, 71, 102, 103, 135, total - 1, total]
        lims = np.array([edges[i % len(edges)] for i in range(40)], np.int32)
        out, lse = run_link(dw.store, cfg, p.chunk_offsets, wl.link_ids(), p.q_offsets, None,
                            wl.q, None, None, lims=lims)
        links = oracle.workload_links(wl, dw.chunks)
        ref, ref_lse = ref_link(cfg, links, wl.q, p.q_offsets, lims=lims)
        bad = G.failures(G.F32 if dtype == W.F32 else G.BF16, out, ref, lse, ref_lse)
        assert not bad, bad
    finally:
        dw.close()


@pytest.mark.parametrize("dtype", [W.F32, W.BF16])
def test_stream_max_jumps(dtype):
    """Scores whose maximum grows by far more than 2^64 from tile to tile, so
    the running max moves again and again, and rows far below it."""
    cfg = W.small_config("stream_jumps", dtype=dtype, d_k=64, n_q_heads=6, n_kv_heads=2,
                         chunk_lens=(200, 200), batch=1, links=(2, 2), q_len=30, self_len=30)
    wl = W.make_workload(cfg)
    # keys scaled by powers of two (exact in both types), growing along each chunk
    grow = (2.0 ** (np.arange(200) // 24)).astype(np.float32)[:, None, None]
    store = pic.Store(cfg.kind, cfg.dtype, cfg.n_kv_heads, 64, 64, 512)
    chunks = {}
    try:
        for c in wl.used_chunks():
            k, v = W.make_chunk(cfg, int(c))
            k = k * grow if dtype == W.F32 else W.f32_to_bf16_bits(W.bf16_bits_to_f32(k) * grow)
            chunks[int(c)] = (k, v)
            store.put(int(wl.chunk_ids[c]), 200, runner.to_device(k, "cuda"),
                      runner.to_device(v, "cuda"), cur_stream())
        p = wl.plan
        out, lse = run_link(store, cfg, p.chunk_offsets, wl.link_ids(), p.q_offsets,
                            p.self_offsets, wl.q, wl.k_self, wl.v_self)
        ref, ref_lse = oracle.run_workload(wl, chunks)
    finally:
        store.close()
    # a score of size s carries fp32 rounding of about d * 2^-24 s, and the
    # output a relative error of that size: scores reach 2^8 * 8 sigma
    smax = np.abs(ref_lse).max()
    tol = 64 * 2.0 ** -24 * smax + (2.0 ** -8 if dtype == W.BF16 else 0)
    assert np.linalg.norm(out - ref) <= tol * np.linalg.norm(ref)
    assert np.abs(lse - ref_lse).max() <= 64 * 2.0 ** -24 * smax + 1e-4
