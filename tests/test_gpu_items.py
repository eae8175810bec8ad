"""Batches cut into a different number of pieces per request, at the sizes
where the cutting, the work mapping or the merge can go wrong: one long
request among short and empty ones, requests without query rows, piece
boundaries on links and inside the own KV, own KV read in place by the decode
kernel around its tile and limit, few (request, kv head) units over many row
blocks, MLA runs of row blocks that do not fill an XCD's share, and the
no-alloc entry's charge. All against the fp64 oracle to the parity bar."""
import math

import numpy as np
import pytest
import torch

from paper_2602_01519_amd import pic
from paper_2602_01519_amd import workloads as W

from test_gpu_link import run_and_check

pytestmark = pytest.mark.gpu

MLA = dict(kind=W.MLA, n_q_heads=16, d_k=576, d_v=512, q_std=1.0, scale=1 / math.sqrt(192))
LENS = (70, 64, 1, 700, 333)
LONG = [3, 3, 4, 3, 0, 3, 4, 1, 3]      # 4000 linked rows, cut many times


def uneven(name, q, own, **kw):
    return W.small_config(name, chunk_lens=LENS, batch=len(q), links=(0, 0), q_len=q, self_len=own,
                          **kw)


CASES = {
    # (config, links per request)
    "prefill_uneven": (uneven("prefill_uneven", (30, 1, 5, 0, 17), (30, 70, 5, 0, 200), d_k=128),
                       [LONG, [2], [], [3], [0, 1]]),
    "prefill_cross": (uneven("prefill_cross", (64, 3, 2, 9), None, d_k=128),
                      [LONG, [], [4, 3], [1]]),
    "stream_uneven_f32": (uneven("stream_uneven_f32", (60, 1, 5, 0, 130), (60, 70, 5, 0, 200),
                                 d_k=64, dtype=W.F32, n_q_heads=6),
                          [LONG, [2], [], [3], [0, 1]]),
    "stream_uneven_bf16": (uneven("stream_uneven_bf16", (90, 1, 5, 0, 130, 2, 2, 2, 2),
                                  (90, 70, 5, 0, 200, 2, 2, 2, 33), d_k=64),
                           [LONG, [2], [], [3], [0, 1], [1], [3], [4], [0]]),
    "mla_uneven": (uneven("mla_uneven", (40, 1, 5, 0, 9), (40, 70, 5, 0, 200), **MLA),
                   [LONG, [2], [], [3], [0, 1]]),
    "mla_decode_uneven": (uneven("mla_decode_uneven", (1, 2, 1, 1), (1, 70, 33, 1), decode=True,
                                 **MLA), [LONG, [2], [], [3, 4]]),
    # one kv head, 8 x 300 rows: the row blocks of one unit spread over the XCDs
    "spread": (uneven("spread", (300,), (300,), d_k=128, n_q_heads=8, n_kv_heads=1), [[3, 4, 0]]),
    "spread_uneven": (uneven("spread_uneven", (200, 3, 70), (210, 3, 70), d_k=128, n_q_heads=24,
                             n_kv_heads=3), [[3, 4], [0], LONG]),
    # a batch of like requests: contiguous row blocks per XCD
    "mla_even": (uneven("mla_even", (4,) * 8, (4,) * 8, **MLA), [[3, 4]] * 8),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_uneven_batches(name):
    cfg, links = CASES[name]
    run_and_check(cfg, links=links)


@pytest.mark.parametrize("own", [1, 31, 32, 33, 63, 64, 65, 127, 128, 129])
@pytest.mark.parametrize("splits", [0, 7])
def test_decode_own_in_place(own, splits):
    """Own KV around the decode kernel's 32-key tiles and around the most it
    reads in place (128 tokens), beside requests with other lengths and
    none linked; 1, 2 and 4 query tokens (causal inside the own tiles)."""
    q = (1, 2, 4, 1)
    cfg = uneven(f"own_{own}", q, tuple(max(a, b) for a, b in zip(q, (own, own, own, 5))), d_k=128,
                 n_q_heads=8, n_kv_heads=2, decode=True)
    run_and_check(cfg, num_splits=splits, links=[[3, 0], [], [4], LONG])


def test_noalloc_charge_is_the_uniform_layout():
    """A call is refused by what the uniform layout of its own KV and partials
    would take, also where the kernels need less: 4 requests of 16 tokens x
    128 heads x 250 splits of 128-wide partials are 1.1 GB, refused, outputs
    untouched; 1 split is accepted."""
    store = pic.Store(W.GQA, W.BF16, 8, 128, 128, 64)
    try:
        k = torch.randn(64, 8, 128, device="cuda").bfloat16()
        store.put(1, 64, k, k)
        B, q, hq = 4, 16, 128
        qo = np.arange(B + 1, dtype=np.int32) * q
        co = np.arange(B + 1, dtype=np.int32)
        qt = torch.randn(B * q, hq, 128, device="cuda").bfloat16()
        out = torch.full((B * q, hq, 128), 7.0, device="cuda", dtype=torch.bfloat16)
        args = (store, co, [1] * B, qo, None, hq, qt, None, None, 1.0, out)
        with pytest.raises(pic.PicError) as e:
            pic.link_decode_noalloc(*args, num_splits=250)
        assert e.value.status == pic.ERR_INVALID
        torch.cuda.synchronize()
        assert bool((out == 7.0).all())
        pic.link_decode_noalloc(*args, num_splits=1)
        torch.cuda.synchronize()
        assert not bool((out == 7.0).all())
    finally:
        store.close()
