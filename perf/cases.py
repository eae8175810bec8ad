"""The work that programs have this library do, as cases for performance measurement.

Every case is a pass through the public entry points of paper_2602_01519_amd.pic, from one
latency-bound question to the largest batch:

  link        prefill-shaped link attention of a batch (pic_link_attn)
  decode      one decode step of a batch (pic_link_decode)
  plan        one decode step through all cross-attention layers of a link plan
  mla         an MLA attention block: query absorption, link attention on the latent
              rows, value up-projection; prefill- or decode-shaped
  blend       a request with recomputed tokens: an uncached document is put, every
              document is derived, the recomputed rows are written layer by layer, the
              recomputed tokens attend under per-query limits, the question attends to
              the derived documents, and the chunks of the request are removed

A case is a dict of plain values (see _DEFAULTS). Its ragged sizes (chunk lengths, links
and tokens per request) come from its own "shape" number, so that they are part of the
case; all tensor values come from the seed.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

from paper_2602_01519_amd import pic

_DEFAULTS = {
    "flow": "link",
    "dtype": "bf16",
    "hq": 32, "hkv": 8, "d": 128,      # GQA heads and width (MLA: hq only, 576 / 512 wide)
    "batch": 1,
    "chunks": 64,                      # chunks the requests choose from
    "len_lo": 512, "len_hi": 512,      # tokens per chunk
    "links_lo": 1, "links_hi": 1,      # links per request
    "disjoint": False,                 # no chunk is linked by two requests
    "q_lo": 1, "q_hi": 1,              # query tokens per request
    "own": True,                       # requests carry own KV
    "own_extra": 0,                    # own tokens before the query tokens
    "starts": False,                   # links skip the first 64 tokens of chunks longer than that
    "layers": 1,
    "prepared": False,                 # arguments marshalled once (PreparedCall)
    "share": 0.0,                      # blend: recomputed share of a document's tokens
    "shape": 1,
}


def _case(name=None, **kw):
    c = dict(_DEFAULTS)
    c.update(kw)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # The smallest fp32 request: 4 links of 128 tokens, 32 question tokens, arguments
        # marshalled once, as a serving loop repeats it. Latency and launches.
        _case("tiny_f32", dtype="f32", hq=8, hkv=2, d=64, chunks=16, len_lo=128, len_hi=128,
              links_lo=4, links_hi=4, q_lo=32, q_hi=32, prepared=True),
        # One question of a few dozen tokens over ten ragged documents: the time to first
        # token of a single interactive user.
        _case("question", chunks=16, len_lo=200, len_hi=1100, links_lo=10, links_hi=10, q_lo=37,
              q_hi=37, shape=2),
        # A batch of such questions over private long documents (the regime the method is
        # made for): bound by reading the linked KV.
        _case("skinny_rag", batch=32, chunks=512, len_lo=1024, len_hi=1024, links_lo=4,
              links_hi=16, disjoint=True, q_lo=16, q_hi=48, shape=3),
        # Batched prefill with the head shape of an 8B GQA backbone, shared documents.
        _case("llama_prefill", batch=8, chunks=64, links_lo=10, links_hi=10, q_lo=256, q_hi=256,
              shape=4),
        # The largest: 16 requests with 8..20 documents of 1024 tokens, 512 query tokens.
        _case("long_rag", batch=16, chunks=256, len_lo=1024, len_hi=1024, links_lo=8,
              links_hi=20, q_lo=512, q_hi=512, shape=5),
        # One decode step of a full batch, 16 private documents each.
        _case("decode", flow="decode", batch=64, chunks=1024, len_lo=1024, len_hi=1024,
              links_lo=16, links_hi=16, disjoint=True, own_extra=127, shape=6),
        # One decode step of a small ragged batch through the eight cross-attention layers
        # of a link plan made once: short kernels, launches and gaps.
        _case("plan_step", flow="plan", batch=6, chunks=40, len_lo=150, len_hi=900, links_lo=2,
              links_hi=9, own_extra=40, layers=8, shape=7),
        # MLA attention block, prefill.
        _case("mla_prefill", flow="mla", hq=16, batch=8, chunks=64, links_lo=12, links_hi=12,
              q_lo=256, q_hi=256, shape=8),
        # MLA attention block, one decode step of a batch.
        _case("mla_decode", flow="mla_decode", hq=16, batch=32, chunks=256, len_lo=300,
              len_hi=1024, links_lo=4, links_hi=14, own_extra=63, shape=9),
        # fp32 caches, a batch of ragged requests whose links skip recomputed first tokens.
        _case("batch_f32", dtype="f32", hq=8, hkv=2, d=64, batch=12, chunks=48, len_lo=100,
              len_hi=700, links_lo=3, links_hi=10, q_lo=20, q_hi=130, starts=True, shape=10),
        # bf16 with 64-wide heads, a batch of ragged requests.
        _case("narrow_heads", hq=32, hkv=8, d=64, batch=8, chunks=64, len_lo=100, len_hi=1000,
              links_lo=4, links_hi=12, q_lo=30, q_hi=300, shape=11),
        # Recomputed tokens (15% of every document) through four layers, then the question.
        _case("blend", flow="blend", batch=2, chunks=12, len_lo=300, len_hi=700, links_lo=5,
              links_hi=6, disjoint=True, q_lo=20, q_hi=50, layers=4, share=0.15, shape=12),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.5)))))))


def _span(rng, lo, hi):
    a, b = sorted((_log_int(rng, lo, hi), _log_int(rng, lo, hi)))
    return a, b


def draw(rng):
    """One more case of the listed ranges, no more work than the largest listed case."""
    most = max(work(c)["flops"] for c in listed())
    while True:
        flow = rng.choice(["link", "link", "link", "decode", "plan", "mla", "mla_decode", "blend"])
        dtype = rng.choice(["bf16", "bf16", "f32"]) if flow in ("link", "decode") else "bf16"
        d = 128 if flow in ("plan", "blend") else rng.choice([64, 128] if dtype == "bf16" else [32, 64])
        hkv = rng.choice([1, 2, 3, 4, 8])
        hq = hkv * rng.choice([1, 2, 4, 5, 8])
        if flow in ("mla", "mla_decode"):
            hkv, hq = 1, rng.choice([8, 16, 16, 20])
        len_lo, len_hi = _span(rng, 64, 1100)
        links_lo, links_hi = _span(rng, 1, 20)
        q_lo, q_hi = _span(rng, 1, 512)
        batch = _log_int(rng, 1, 64)
        kw = dict(flow=flow, dtype=dtype, hq=hq, hkv=hkv, d=d, len_lo=len_lo, len_hi=len_hi,
                  shape=rng.randrange(1 << 20))
        if flow in ("decode", "plan", "mla_decode"):
            q_lo = q_hi = 1
            kw["own_extra"] = _log_int(rng, 1, 200)
        if flow == "link":
            kw["own"] = rng.random() < 0.8
            kw["starts"] = rng.random() < 0.3
            kw["prepared"] = rng.random() < 0.3
        if flow == "plan":
            kw["layers"] = rng.randint(2, 8)
            batch = _log_int(rng, 1, 16)
        if flow == "blend":
            kw.update(layers=rng.randint(1, 4), share=round(rng.uniform(0.02, 0.25), 3))
            batch, links_hi = rng.randint(1, 3), min(links_hi, 6)
            links_lo = min(links_lo, links_hi)
            q_lo, q_hi = min(q_lo, 60), min(q_hi, 60)
        disjoint = flow == "blend" or rng.random() < 0.4
        kw.update(batch=batch, links_lo=links_lo, links_hi=links_hi, q_lo=q_lo, q_hi=q_hi,
                  disjoint=disjoint,
                  chunks=batch * links_hi if disjoint else links_hi + _log_int(rng, 1, 200))
        c = _case(**kw)
        w = work(c)
        if 2e6 < w["flops"] <= most and w["bytes"] <= 4.4e9 and \
                c["chunks"] * c["len_hi"] * c["layers"] * _token_bytes(c) <= 6e9:
            return c


# ---------------------------------------------------------------------------
# Shapes of a case

def _is_mla(c):
    return c["flow"] in ("mla", "mla_decode")


def _widths(c):
    return (576, 512) if _is_mla(c) else (c["d"], c["d"])


def _esize(c):
    return 4 if c["dtype"] == "f32" else 2


def _token_bytes(c):
    d_k, d_v = _widths(c)
    return _esize(c) * (d_k if _is_mla(c) else c["hkv"] * (d_k + d_v))


class _Shape:
    """Chunk lengths, links and token counts of a case."""

    def __init__(self, c):
        r = random.Random(c["shape"])
        self.lens = [r.randint(c["len_lo"], c["len_hi"]) for _ in range(c["chunks"])]
        counts = [r.randint(c["links_lo"], c["links_hi"]) for _ in range(c["batch"])]
        if c["disjoint"]:
            perm = list(range(c["chunks"]))
            r.shuffle(perm)
            self.links = [[perm.pop() for _ in range(n)] for n in counts]
        else:
            self.links = [r.sample(range(c["chunks"]), n) for n in counts]
        self.q = [r.randint(c["q_lo"], c["q_hi"]) for _ in range(c["batch"])]
        self.own = [n + c["own_extra"] if c["own"] else 0 for n in self.q]
        self.start = [64 if c["starts"] and n > 64 else 0 for n in self.lens]
        self.used = sorted({i for l in self.links for i in l})
        # blend: the recomputed rows of every linked document
        self.rows = {}
        if c["flow"] == "blend":
            for i in self.used:
                n = max(1, int(round(c["share"] * self.lens[i])))
                self.rows[i] = sorted(r.sample(range(self.lens[i]), n))

    def doc(self, r):
        return sum(self.lens[i] - self.start[i] for i in self.links[r])

    def pairs(self, r):
        """Visible (query token, key) pairs of request r."""
        own = self.own[r]
        if own == 0:
            return self.q[r] * self.doc(r)
        return self.q[r] * self.doc(r) + sum(i + 1 + own - self.q[r] for i in range(self.q[r]))


def _offsets(counts):
    return np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)


def _chunk_id(i):
    return 0x5851F42D4C957F2D * (i + 1) & 0x7FFFFFFFFFFFFFFF


def work(case):
    """Bytes and operations of one pass: linked KV, own KV and queries read once, outputs
    written once, visible pairs only."""
    c, s = case, _Shape(case)
    d_k, d_v = _widths(c)
    es, hq, layers = _esize(c), c["hq"], c["layers"]
    tq, ts = sum(s.q), sum(s.own)
    kv = sum(s.lens[i] - s.start[i] for i in s.used) * _token_bytes(c) * layers
    pairs = sum(s.pairs(r) for r in range(c["batch"]))
    bytes_ = kv + layers * (ts * _token_bytes(c) + tq * hq * 4)
    flops = layers * pairs * hq * 2 * (d_k + d_v)
    if _is_mla(c):
        bytes_ += tq * hq * (192 + 128) * es + 2 * hq * 128 * 512 * es
        flops += tq * hq * 4 * 128 * 512
    else:
        bytes_ += layers * tq * hq * (d_k + d_v) * es
    if c["flow"] == "blend":
        tr = sum(len(v) for v in s.rows.values())
        cold = s.lens[s.links[0][0]]
        # recomputed rows read and written, their queries and outputs; the uncached
        # document read and written
        bytes_ += layers * (2 * tr * _token_bytes(c) + tr * hq * ((d_k + d_v) * es + 4) +
                            2 * cold * _token_bytes(c))
        seen = sum(_limits(s, r).sum() for r in range(c["batch"]))
        flops += layers * int(seen) * hq * 2 * (d_k + d_v)
    return {"bytes": float(bytes_), "flops": float(flops)}


def _limits(s, r):
    """blend: linked rows the recomputed tokens of request r see (position + 1)."""
    out, base = [], 0
    for i in s.links[r]:
        out += [base + t + 1 for t in s.rows[i]]
        base += s.lens[i]
    return np.array(out, dtype=np.int32)


def tolerance(case):
    # Four times what the present code shows against 64 bits. bf16: probabilities and
    # outputs are rounded to 8 significant bits; the MLA block rounds the absorbed query
    # and the latent output too. fp32: sums in another order.
    if case["dtype"] == "f32":
        return {"rel": 2e-6}
    return {"rel": 1.2e-2 if _is_mla(case) else 1e-2}


# ---------------------------------------------------------------------------
# Inputs

class _Draw:
    """Seeded N(0, 1) tensors in the case's dtype, one after another."""

    def __init__(self, c, seed):
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(seed * 1000003 + c["shape"])
        self.dtype = torch.float32 if c["dtype"] == "f32" else torch.bfloat16

    def __call__(self, *shape, std=1.0):
        x = torch.randn(shape, generator=self.gen, device="cuda", dtype=torch.float32)
        return (x * std if std != 1.0 else x).to(self.dtype)


def _chunk(c, s, rnd, i):
    """(k, v) of chunk i, [layers][tokens][heads][width], v None for MLA."""
    d_k, d_v = _widths(c)
    hkv = 1 if _is_mla(c) else c["hkv"]
    k = rnd(c["layers"], s.lens[i], hkv, d_k)
    return k, None if _is_mla(c) else rnd(c["layers"], s.lens[i], hkv, d_v)


def _q_std(c):
    # scores of order one: bf16 GQA folds 1/sqrt(d) into the query, as the scale is 1
    return 1.0 / math.sqrt(c["d"]) if c["dtype"] == "bf16" and not _is_mla(c) else 1.0


def _scale(c):
    if _is_mla(c):
        return 1.0 / math.sqrt(192.0)
    return 1.0 if c["dtype"] == "bf16" else 1.0 / math.sqrt(c["d"])


def _tensors(c, s, rnd):
    """Per-request inputs (after the chunks): queries, own KV, weights, recomputed rows."""
    d_k, d_v = _widths(c)
    tq, ts, layers = sum(s.q), sum(s.own), c["layers"]
    t = {}
    if _is_mla(c):
        t["q"] = rnd(tq, c["hq"], 192)
        t["w_uk"] = rnd(c["hq"], 512, 128, std=0.5 / math.sqrt(128.0))
        t["w_uv"] = rnd(c["hq"], 128, 512, std=1.0 / math.sqrt(512.0))
        t["k"] = rnd(1, ts, 1, d_k)
        t["v"] = None
        return t
    t["q"] = rnd(layers, tq, c["hq"], d_k, std=_q_std(c))
    t["k"] = rnd(layers, ts, c["hkv"], d_k) if ts else None
    t["v"] = rnd(layers, ts, c["hkv"], d_v) if ts else None
    if c["flow"] == "blend":
        tr = sum(len(v) for v in s.rows.values())
        t["rq"] = rnd(layers, tr, c["hq"], d_k, std=_q_std(c))
        t["rows"] = {i: (rnd(layers, len(s.rows[i]), c["hkv"], d_k),
                         rnd(layers, len(s.rows[i]), c["hkv"], d_v)) for i in s.used}
    return t


def _stream():
    return torch.cuda.current_stream().cuda_stream


class _State:
    pass


def prepare(case, seed):
    c, s = case, _Shape(case)
    d_k, d_v = _widths(c)
    rnd = _Draw(c, seed)
    cold = s.links[0][0] if c["flow"] == "blend" else None
    pages = sum((s.lens[i] + 63) // 64 * 64 for i in s.used)
    if c["flow"] == "blend":
        pages *= 6                      # derived pages of a few requests in flight
    st = _State()
    st.c, st.s = c, s
    st.store = pic.Store(pic.MLA if _is_mla(c) else pic.GQA,
                         pic.F32 if c["dtype"] == "f32" else pic.BF16,
                         1 if _is_mla(c) else c["hkv"], d_k, d_v, pages, n_layers=c["layers"])
    for i in s.used:
        k, v = _chunk(c, s, rnd, i)
        if i == cold:
            st.cold = (_chunk_id(i), k.shape[1], k, v)
        else:
            st.store.put(_chunk_id(i), k.shape[1], k, v, _stream())
    st.t = _tensors(c, s, rnd)
    st.offsets = _offsets([len(l) for l in s.links])
    index = [i for l in s.links for i in l]
    st.ids = np.array([_chunk_id(i) for i in index], dtype=np.uint64)
    st.q_offsets = _offsets(s.q)
    st.own_offsets = _offsets(s.own) if c["own"] else None
    st.starts = np.array([s.start[i] for i in index], dtype=np.int32) if c["starts"] else None
    st.scale = float(np.float32(_scale(c)))
    tq, layers = sum(s.q), c["layers"]
    st.out = torch.empty(layers, tq, c["hq"], d_v, dtype=rnd.dtype, device="cuda")
    st.lse = torch.empty(layers, tq, c["hq"], dtype=torch.float32, device="cuda")
    t = st.t
    if _is_mla(c):
        st.q_abs = torch.empty(tq, c["hq"], 576, dtype=rnd.dtype, device="cuda")
        st.up = torch.empty(tq, c["hq"], 128, dtype=rnd.dtype, device="cuda")
    elif c["flow"] == "plan":
        st.plan = pic.LinkPlan(st.store, st.offsets, st.ids, st.q_offsets, st.own_offsets,
                               c["hq"], mode=pic.DECODE)
    elif c["flow"] == "blend":
        st.derived = {i: _chunk_id(i + c["chunks"]) for i in s.used}
        st.der_ids = np.array([st.derived[i] for i in index], dtype=np.uint64)
        st.row_list = {i: np.array(s.rows[i], dtype=np.int32) for i in s.used}
        st.rec_offsets = _offsets([sum(len(s.rows[i]) for i in l) for l in s.links])
        st.limits = np.concatenate([_limits(s, r) for r in range(c["batch"])])
        tr = int(st.rec_offsets[-1])
        st.rec_out = torch.empty(layers, tr, c["hq"], d_v, dtype=rnd.dtype, device="cuda")
        st.rec_lse = torch.empty(layers, tr, c["hq"], dtype=torch.float32, device="cuda")
    elif c["prepared"]:
        st.call = pic.PreparedCall(c["flow"] == "decode", st.store, st.offsets, st.ids,
                                   st.q_offsets, st.own_offsets, c["hq"], t["q"], t["k"], t["v"],
                                   st.scale, st.out, st.lse, chunk_starts=st.starts)
    return st


def run(st):
    c, t, stream = st.c, st.t, _stream()
    if _is_mla(c):
        tq = t["q"].shape[0]
        pic.mla_absorb_q(tq, c["hq"], t["q"], t["w_uk"], st.q_abs, stream)
        link = pic.link_decode if c["flow"] == "mla_decode" else pic.link_attn
        link(st.store, st.offsets, st.ids, st.q_offsets, st.own_offsets, c["hq"], st.q_abs, t["k"],
             None, st.scale, st.out, st.lse, stream=stream)
        pic.mla_up_v(tq, c["hq"], st.out, t["w_uv"], st.up, stream)
        return st.q_abs, st.out, st.lse, st.up
    if c["flow"] == "plan":
        for l in range(c["layers"]):
            st.plan.run(l, t["q"][l], t["k"][l], t["v"][l], st.scale, st.out[l], st.lse[l],
                        stream=stream)
        return st.out, st.lse
    if c["flow"] == "blend":
        return _run_blend(st, stream)
    if c["prepared"]:
        st.call(stream)
    else:
        link = pic.link_decode if c["flow"] == "decode" else pic.link_attn
        link(st.store, st.offsets, st.ids, st.q_offsets, st.own_offsets, c["hq"], t["q"], t["k"],
             t["v"], st.scale, st.out, st.lse, stream=stream, chunk_starts=st.starts)
    return st.out, st.lse


def _run_blend(st, stream):
    c, t, store = st.c, st.t, st.store
    store.put(*st.cold, stream)
    for i in st.s.used:
        store.derive(st.derived[i], _chunk_id(i), st.row_list[i], stream)
    for l in range(c["layers"]):
        for i in st.s.used:
            k, v = t["rows"][i]
            store.write_rows(st.derived[i], l, st.row_list[i], k[l], v[l], stream)
        pic.link_attn(store, st.offsets, st.der_ids, st.rec_offsets, None, c["hq"], t["rq"][l],
                      None, None, st.scale, st.rec_out[l], st.rec_lse[l], stream=stream, layer=l,
                      q_doc_limits=st.limits)
        pic.link_attn(store, st.offsets, st.der_ids, st.q_offsets, st.own_offsets, c["hq"],
                      t["q"][l], t["k"][l], t["v"][l], st.scale, st.out[l], st.lse[l],
                      stream=stream, layer=l)
    for i in st.s.used:
        store.remove(st.derived[i], stream)
    store.remove(st.cold[0], stream)
    return st.rec_out, st.rec_lse, st.out, st.lse


# ---------------------------------------------------------------------------
# The same in 64 bits, plain torch

def _attend(q, keys, values, scale, n_kv, limit):
    """q [rows][hq][d_k] over keys / values [n][n_kv][..]; row i sees the keys below
    limit[i] (a tensor of row limits, or a (rows, keys) mask). Returns (out, lse)."""
    rows, hq, _ = q.shape
    group = hq // n_kv
    out = torch.empty(rows, hq, values.shape[2], dtype=torch.float64, device="cuda")
    lse = torch.empty(rows, hq, dtype=torch.float64, device="cuda")
    for h in range(n_kv):
        k, v = keys[:, h].double(), values[:, h].double()
        step = max(1, (1 << 27) // max(1, k.shape[0] * group))
        for a in range(0, rows, step):
            part = q[a:a + step, h * group:(h + 1) * group].double()
            n = part.shape[0]
            x = part.reshape(n * group, -1) @ k.t() * scale
            hide = ~limit[a:a + n].repeat_interleave(group, 0)
            x.masked_fill_(hide, -math.inf)
            m = x.max(1, keepdim=True).values
            x = torch.exp_(x - m)
            z = x.sum(1, keepdim=True)
            out[a:a + n, h * group:(h + 1) * group] = (x @ v / z).reshape(n, group, -1)
            lse[a:a + n, h * group:(h + 1) * group] = (m + z.log()).reshape(n, group)
    return out, lse


def _visible(n_doc, lq, ls):
    """(lq, n_doc + ls) mask: every linked row, own rows up to the token itself."""
    own = torch.arange(ls, device="cuda")[None, :] <= \
        torch.arange(lq, device="cuda")[:, None] + (ls - lq)
    return torch.cat([torch.ones(lq, n_doc, dtype=torch.bool, device="cuda"), own], 1)


def exact(case, seed):
    c, s = case, _Shape(case)
    d_k, d_v = _widths(c)
    rnd = _Draw(c, seed)
    chunks = {i: _chunk(c, s, rnd, i) for i in s.used}
    t = _tensors(c, s, rnd)
    q_off, own_off = _offsets(s.q), _offsets(s.own)
    scale = float(np.float32(_scale(c)))
    hkv = 1 if _is_mla(c) else c["hkv"]
    if _is_mla(c):
        nope, rope = t["q"][..., :128].double(), t["q"][..., 128:].double()
        q_abs = torch.cat([torch.stack([nope[:, h] @ t["w_uk"][h].double().t()
                                        for h in range(c["hq"])], 1), rope], 2)
    outs, lses, recs = [], [], []
    for l in range(c["layers"]):
        out = torch.empty(sum(s.q), c["hq"], d_v, dtype=torch.float64, device="cuda")
        lse = torch.empty(sum(s.q), c["hq"], dtype=torch.float64, device="cuda")
        rec = []
        for r in range(c["batch"]):
            ks, vs = [], []
            for i in s.links[r]:
                k, v = chunks[i]
                k, v = k[l], (k[l, :, :, :d_v] if v is None else v[l])
                if c["flow"] == "blend":
                    at = torch.tensor(s.rows[i], device="cuda")
                    k, v = k.clone(), v.clone()
                    k[at], v[at] = t["rows"][i][0][l], t["rows"][i][1][l]
                ks.append(k[s.start[i]:])
                vs.append(v[s.start[i]:])
            n_doc = s.doc(r)
            if c["flow"] == "blend":
                lim = torch.tensor(_limits(s, r), device="cuda")
                a = sum(x[0].shape[0] for x in rec)
                see = torch.arange(n_doc, device="cuda")[None, :] < lim[:, None]
                rec.append(_attend(t["rq"][l][a:a + len(lim)], torch.cat(ks), torch.cat(vs), scale,
                                   hkv, see))
            if s.own[r]:
                own = t["k"][l, own_off[r]:own_off[r + 1]]
                ks.append(own)
                vs.append(own[:, :, :d_v] if t["v"] is None else
                          t["v"][l, own_off[r]:own_off[r + 1]])
            q = (q_abs if _is_mla(c) else t["q"][l])[q_off[r]:q_off[r + 1]]
            o, z = _attend(q, torch.cat(ks), torch.cat(vs), scale, hkv,
                           _visible(n_doc, s.q[r], s.own[r]))
            out[q_off[r]:q_off[r + 1]], lse[q_off[r]:q_off[r + 1]] = o, z
        outs.append(out)
        lses.append(lse)
        recs.append(rec)
    out, lse = torch.stack(outs), torch.stack(lses)
    if _is_mla(c):
        up = torch.stack([out[0, :, h] @ t["w_uv"][h].double().t() for h in range(c["hq"])], 1)
        return q_abs, out, lse, up
    if c["flow"] == "blend":
        return (torch.stack([torch.cat([x[0] for x in rec]) for rec in recs]),
                torch.stack([torch.cat([x[1] for x in rec]) for rec in recs]), out, lse)
    return out, lse
