"""Batches cut into a different number of pieces per request, at the sizes
where the cutting, the work mapping or the merge can go wrong: one long
request among short and empty ones, requests without query rows, piece
boundaries on links and inside the own KV, own KV read in place by the decode
kernel around its tiles and long, few (request, kv head) units over many row
blocks, MLA runs of row blocks that do not fill an XCD's share, and the
no-alloc entry's charge. All against the fp64 oracle to the parity bar."""
import dataclasses
import math

import numpy as np
import pytest
import torch

import oracle
import parity_gate as G
from paper_2602_01519_amd import pic, runner
from paper_2602_01519_amd import workloads as W

from test_gpu_blend import ref_link, run_link
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
    """Own KV, which the decode kernel reads in place, around its 32-key tiles,
    beside requests with other lengths and none linked; 1, 2 and 4 query
    tokens (causal inside the own tiles)."""
    q = (1, 2, 4, 1)
    cfg = uneven(f"own_{own}", q, tuple(max(a, b) for a, b in zip(q, (own, own, own, 5))), d_k=128,
                 n_q_heads=8, n_kv_heads=2, decode=True)
    run_and_check(cfg, num_splits=splits, links=[[3, 0], [], [4], LONG])


@pytest.mark.parametrize("own,splits", [(513, 0), (3000, 0), (3000, 7), (4097, 100)])
def test_decode_long_own(own, splits):
    """Own KV longer than the documents, cut into pieces of its own, on both the
    call and a plan's run (the same bits)."""
    q = (1, 2, 4, 1)
    cfg = uneven(f"long_own_{own}", q, (own, own + 1, 4, own - 1), d_k=128, n_q_heads=8,
                 n_kv_heads=2, decode=True)
    links = [[3, 0], [], [4], [1]]
    out, lse = run_and_check(cfg, num_splits=splits, links=links)
    wl = W.make_workload(cfg)
    p = wl.plan
    idx = np.array([c for l in links for c in l], dtype=np.int64)
    co = np.cumsum([0] + [len(l) for l in links]).astype(np.int32)
    dw = runner.upload(dataclasses.replace(wl, plan=dataclasses.replace(
        p, chunk_offsets=co, chunk_index=idx)))
    try:
        plan = pic.LinkPlan(dw.store, co, wl.chunk_ids[idx], p.q_offsets, p.self_offsets,
                            cfg.n_q_heads, mode=pic.DECODE, num_splits=splits)
        plan.run(0, dw.q, dw.k_self, dw.v_self, float(np.float32(cfg.scale)), dw.out, dw.lse,
                 stream=torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        a, la = dw.results()
        plan.close()
        assert np.array_equal(a, out) and np.array_equal(la, lse)
    finally:
        dw.close()


def test_noalloc_charge_is_the_uniform_layout():
    """A call is refused by what the uniform layout of its own KV and partials
    would take: 4 requests of 16 tokens x 128 heads x 250 splits of 128-wide
    partials are 1.1 GB, refused, outputs untouched; 1 split is accepted; 40
    one-token requests of 2000 own tokens are refused for 164 MB of own KV,
    which the decode kernel would read in place."""
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
        n, own = 40, 2000
        one = np.arange(n + 1, dtype=np.int32)
        ks = torch.zeros(n * own, 8, 128, device="cuda", dtype=torch.bfloat16)
        out = torch.full((n, 32, 128), 7.0, device="cuda", dtype=torch.bfloat16)
        with pytest.raises(pic.PicError) as e:
            pic.link_decode_noalloc(store, one, [1] * n, one, one * own, 32, qt[:n, :32].contiguous(),
                                    ks, ks, 1.0, out)
        assert e.value.status == pic.ERR_INVALID
        torch.cuda.synchronize()
        assert bool((out == 7.0).all())
    finally:
        store.close()


@pytest.mark.parametrize("pattern", ["rising", "falling", "edges", "none_seen"])
def test_limited_row_blocks(pattern):
    """Cross-only calls with per-query limits whose row blocks end at different
    tiles (five 256-row blocks, a split call): rising limits as recomputed
    tokens have, falling ones, limits on tile and link edges, and row blocks
    that see nothing at all."""
    q = (300, 40)
    cfg = uneven("limited", q, None, d_k=128, n_q_heads=8, n_kv_heads=2)
    wl = W.make_workload(cfg)
    links = [LONG, [4, 3]]
    idx = np.array([c for l in links for c in l], dtype=np.int64)
    co = np.array([0, len(links[0]), len(idx)], np.int32)
    rows = [sum(LENS[c] for c in l) for l in links]
    lims = []
    for n, total in zip(q, rows):
        if pattern == "rising":
            lims.append(np.sort(np.random.default_rng(n).integers(1, total + 1, n)))
        elif pattern == "falling":
            lims.append(np.linspace(total, 0, n).astype(int))
        elif pattern == "edges":
            edges = [0, 1, 63, 64, 65, 699, 700, 701, 764, total - 1, total]
            lims.append(np.array([min(edges[i % len(edges)], total) for i in range(n)]))
        else:
            lims.append(np.where(np.arange(n) < 130, 0, total))
    lims = np.concatenate(lims).astype(np.int32)
    dw = runner.upload(dataclasses.replace(wl, plan=dataclasses.replace(
        wl.plan, chunk_offsets=co, chunk_index=idx)))
    try:
        out, lse = run_link(dw.store, cfg, co, wl.chunk_ids[idx], wl.plan.q_offsets, None, wl.q,
                            None, None, lims=lims)
        ref, ref_lse = ref_link(cfg, [[dw.chunks[c] for c in l] for l in links], wl.q,
                                wl.plan.q_offsets, lims=lims)
        bad = G.failures(G.BF16, out, ref, lse, ref_lse)
        assert not bad, bad
    finally:
        dw.close()


@pytest.mark.parametrize("splits", [2, 5, 100])
@pytest.mark.parametrize("d", [64, 128])
def test_limited_empty_pieces(d, splits):
    """Cross-only decode calls with per-query limits cut into more pieces than
    their requests have tiles (3, 1 and 11): the empty pieces, those of the
    table's last link among them, walk no links."""
    q = (16, 4, 9)
    cfg = uneven("limited_empty", q, None, d_k=d, n_q_heads=8, n_kv_heads=2, decode=True)
    wl = W.make_workload(cfg)
    links = [[0, 1], [2], [3]]
    idx = np.array([c for l in links for c in l], dtype=np.int64)
    co = np.array([0, 2, 3, 4], np.int32)
    lims = np.concatenate([np.linspace(0, sum(LENS[c] for c in l), n).astype(int)
                           for l, n in zip(links, q)]).astype(np.int32)
    dw = runner.upload(dataclasses.replace(wl, plan=dataclasses.replace(
        wl.plan, chunk_offsets=co, chunk_index=idx)))
    try:
        out, lse = run_link(dw.store, cfg, co, wl.chunk_ids[idx], wl.plan.q_offsets, None, wl.q,
                            None, None, lims=lims, decode=True, splits=splits)
        ref, ref_lse = ref_link(cfg, [[dw.chunks[c] for c in l] for l in links], wl.q,
                                wl.plan.q_offsets, lims=lims)
        bad = G.failures(G.BF16, out, ref, lse, ref_lse)
        assert not bad, bad
    finally:
        dw.close()


@pytest.mark.parametrize("d,dtype,hq,q,own,decode", [
    (128, W.BF16, 8, 40, None, False), (128, W.BF16, 8, 300, None, False),
    (64, W.BF16, 6, 70, None, False), (64, W.F32, 6, 70, None, False),
    (128, W.BF16, 8, 2, 70, True),                                    # decode kernel, own in place
    (128, W.BF16, 8, 40, 70, False), (64, W.F32, 6, 70, 90, False),   # own laid out
    (64, W.BF16, 6, 20, 50, False), (64, W.F32, 6, 20, 50, False),    # small calls, own in place
    (64, W.BF16, 8, 20, 50, False)])                                  # lean
def test_unaligned_tensors(d, dtype, hq, q, own, decode):
    """Query, own KV and output tensors that start one element past a 16-byte
    boundary give the bits aligned ones give, which match the oracle."""
    cfg = W.small_config("unaligned", dtype=dtype, d_k=d, n_q_heads=hq, n_kv_heads=2,
                         chunk_lens=(700, 130), batch=1, links=(2, 2), q_len=q, self_len=own,
                         decode=decode)
    wl = W.make_workload(cfg)
    p = wl.plan
    dw = runner.upload(wl)
    n = dw.out.numel()

    def shifted(t, off):
        if t is None:
            return None
        buf = torch.zeros(t.numel() + 8, dtype=t.dtype, device="cuda")
        buf[off:off + t.numel()] = t.reshape(-1)
        return buf[off:]

    try:
        outs = []
        for off in (0, 1):
            res = torch.zeros(n + 8, dtype=dw.out.dtype, device="cuda")
            lse = torch.zeros(dw.lse.numel(), dtype=torch.float32, device="cuda")
            call = pic.link_decode if decode else pic.link_attn
            call(dw.store, p.chunk_offsets, wl.link_ids(), p.q_offsets, p.self_offsets, hq,
                 shifted(dw.q, off), shifted(dw.k_self, off), shifted(dw.v_self, off),
                 float(np.float32(cfg.scale)), res[off:], lse,
                 stream=torch.cuda.current_stream().cuda_stream)
            torch.cuda.synchronize()
            outs.append((res[off:off + n].clone(), lse))
            assert int((res[:off] != 0).sum()) == 0 and int((res[off + n:] != 0).sum()) == 0
        assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1])
        ref, ref_lse = oracle.run_workload(wl, dw.chunks)
        out = runner.to_host(outs[0][0].reshape(dw.out.shape), dtype)
        bad = G.failures(G.F32 if dtype == W.F32 else G.BF16, out, ref,
                         outs[0][1].reshape(dw.lse.shape).cpu().numpy().astype(np.float64), ref_lse)
        assert not bad, bad
    finally:
        dw.close()


def test_limited_workspace_is_bounded():
    """A limited call whose row blocks walk almost none of its tiles (4095 of
    4096 query tokens see one linked row, the last sees 65,536): empty pieces
    cost next to no time but their rows of partials take memory all the same,
    so the pieces are bounded by it (144 MiB; cutting them by time alone took
    32 pieces and 2.2 GB)."""
    n, links = 4096, 64
    store = pic.Store(W.GQA, W.BF16, 8, 128, 128, 1024)
    try:
        g = torch.Generator(device="cuda").manual_seed(1)
        k = torch.randn(1024, 8, 128, device="cuda", generator=g).bfloat16()
        v = torch.randn(1024, 8, 128, device="cuda", generator=g).bfloat16()
        store.put(1, 1024, k, v)
        q = torch.randn(n, 32, 128, device="cuda", generator=g).bfloat16() / 8
        out = torch.empty_like(q)
        lims = np.ones(n, np.int32)
        lims[-1] = 1024 * links
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        free = torch.cuda.mem_get_info()[0]
        pic.link_attn(store, np.array([0, links], np.int32), [1] * links,
                      np.array([0, n], np.int32), None, 32, q, None, None, 1.0, out,
                      q_doc_limits=lims)
        torch.cuda.synchronize()
        used = free - torch.cuda.mem_get_info()[0]
        assert used <= 160 << 20, used
        # one linked row: its value; the repeated chunk: attention over it once
        want = v[0].repeat_interleave(4, 0).expand(n - 1, -1, -1)
        assert torch.equal(out[:-1], want)
        s = torch.einsum("hd,thd->ht", q[-1].float(), k.float().repeat_interleave(4, 1))
        ref = torch.einsum("ht,thd->hd", s.softmax(1), v.float().repeat_interleave(4, 1))
        assert float((out[-1].float() - ref).norm() / ref.norm()) <= 2.0 ** -7
    finally:
        store.close()
