"""Values at the ends of the fp32 range, and infinities and NaN in the caches.

The streaming kernel of fp32 and narrow bf16 GQA calls keeps its probabilities
at or below one, so sums of values stay finite as long as the values' own sums
do; keys a query row does not see (rows past a limit that cuts a link inside a
page, own keys after the row's token) do not reach its output, whatever they
hold; a visible infinite value gives an infinite output. In every kernel a NaN
score makes the row NaN also where its keys are split over several pieces."""
import math

import numpy as np
import pytest
import torch

from paper_2602_01519_amd import pic, runner
from paper_2602_01519_amd import workloads as W

from test_gpu_blend import ref_link, run_link, stream as cur_stream

pytestmark = pytest.mark.gpu

MLA = dict(kind=W.MLA, n_q_heads=16, d_k=576, d_v=512, q_std=1.0, scale=1 / math.sqrt(192))
# the streaming kernel's shapes (a group of 3 keeps small calls off the lean kernel)
STREAM = [(W.F32, 32), (W.F32, 64), (W.F32, 128), (W.BF16, 32), (W.BF16, 64)]


def narrow(dtype, d, lens, batch, q, own, decode=False, hq=6):
    return W.small_config("range", dtype=dtype, d_k=d, n_q_heads=hq, n_kv_heads=2, chunk_lens=lens,
                          batch=batch, links=(0, 0), q_len=q, self_len=own, decode=decode)


def to_store(cfg, x):
    """fp32 host array in the store's dtype."""
    return W.f32_to_bf16_bits(x) if x is not None and cfg.dtype == W.BF16 else x


def run_calls(cfg, calls, links, q, lims=None, splits=0):
    """Outputs of one call per chunk set in `calls` (each a list of fp32 (k, v, n)), all with
    the same links (chunk numbers per request) and query."""
    co = np.cumsum([0] + [len(l) for l in links]).astype(np.int32)
    ids = np.array([1 + c for l in links for c in l], np.uint64)
    n = q.shape[0] // len(links)
    qo = (np.arange(len(links) + 1) * n).astype(np.int32)
    res = []
    for chunks, own in calls:
        store = pic.Store(cfg.kind, cfg.dtype, cfg.n_kv_heads, cfg.d_k, cfg.d_v,
                          sum((len(k) + 63) // 64 * 64 for k, _ in chunks))
        try:
            for i, (k, v) in enumerate(chunks):
                store.put(1 + i, len(k), runner.to_device(to_store(cfg, k), "cuda"),
                          None if v is None else runner.to_device(to_store(cfg, v), "cuda"),
                          cur_stream())
            so = None
            if own is not None:
                m = own[0].shape[0] // len(links)
                so = (np.arange(len(links) + 1) * m).astype(np.int32)
            res.append(run_link(store, cfg, co, ids, qo, so, to_store(cfg, q),
                                None if own is None else to_store(cfg, own[0]),
                                None if own is None else to_store(cfg, own[1]), lims=lims,
                                decode=cfg.decode, splits=splits))
        finally:
            store.close()
    return res


def normal(rng, *shape):
    return rng.standard_normal(shape, dtype=np.float32)


@pytest.mark.parametrize("batch,splits", [(1, None), (9, None), (1, 0), (9, 3)])
@pytest.mark.parametrize("dtype,d", STREAM)
def test_large_values_stay_finite(dtype, d, batch, splits):
    """Scores that grow by 2^29 from chunk to chunk (20 in natural logs) beside
    values of size 2^110: a probability above one would overflow their sums."""
    rng = np.random.default_rng(d + batch)
    q_len = 2 if splits is not None else 21
    lens = (70, 90, 333)
    cfg = narrow(dtype, d, lens, batch, (q_len,) * batch, None, decode=splits is not None)
    q = 1 + np.float32(0.1) * normal(rng, batch * q_len, 6, d)
    chunks = []
    for i, n in enumerate(lens):
        k = np.float32(0.1) * normal(rng, n, 2, d) + np.float32(10 * i / (cfg.scale * d))
        chunks.append((k, np.float32(2.0 ** 110) * normal(rng, n, 2, d)))
    links = [[0, 1, 2]] * batch
    (out, lse), = run_calls(cfg, [(chunks, None)], links, q, splits=splits or 0)
    unit = [(to_store(cfg, k), to_store(cfg, v * np.float32(2.0 ** -110))) for k, v in chunks]
    qo = (np.arange(batch + 1) * q_len).astype(np.int32)
    ref, ref_lse = ref_link(cfg, [[unit[c] for c in l] for l in links], to_store(cfg, q), qo)
    assert np.isfinite(out).all()
    # a score of size 20 carries fp32 rounding of some 2^-24 x 20, the output the same
    bad = np.linalg.norm(out * 2.0 ** -110 - ref) / np.linalg.norm(ref)
    assert bad <= (2.0 ** -7 if dtype == W.BF16 else 64 * 2.0 ** -24 * 20), bad
    assert np.abs(lse - ref_lse).max() <= 64 * 2.0 ** -24 * 20


def same(cfg, a, b, sel=np.s_[:]):
    """Results of the same sums in another order: fp32 sums of some hundred
    terms, rounded to the store's type."""
    tol = 2.0 ** -8 if cfg.dtype == W.BF16 else 2e-6
    (x, lx), (y, ly) = (a[0][sel], a[1][sel]), (b[0][sel], b[1][sel])
    assert np.isfinite(x).all() and np.isfinite(y).all()
    assert np.linalg.norm(x - y) <= tol * np.linalg.norm(y)
    assert np.abs(lx - ly).max() <= 1e-5


BAD = [math.inf, -math.inf, math.nan]


def spoil(a, rows):
    """A copy of a with the given rows full of infinities and NaN."""
    b = a.copy()
    for i, r in enumerate(rows):
        b[r] = BAD[i % 3]
    return b


@pytest.mark.parametrize("form", ["small", "items", "decode"])
@pytest.mark.parametrize("dtype,d", STREAM)
def test_rows_past_a_uniform_limit(dtype, d, form):
    """Every query row sees 100 of a chunk's 200 rows: the link is cut inside a
    page, whose other rows hold infinities and NaN."""
    rng = np.random.default_rng(d)
    batch, q_len = (9, 7) if form == "items" else (1, 2 if form == "decode" else 30)
    cfg = narrow(dtype, d, (64, 200), batch, (q_len,) * batch, None, decode=form == "decode")
    q = normal(rng, batch * q_len, 6, d) * np.float32(cfg.q_std)
    first = (normal(rng, 64, 2, d), normal(rng, 64, 2, d))
    k, v = normal(rng, 200, 2, d), normal(rng, 200, 2, d)
    lims = np.full(batch * q_len, 164, np.int32)
    hidden = range(100, 200)
    clean, dirty = run_calls(cfg, [([first, (k, v)], None),
                                   ([first, (spoil(k, hidden), spoil(v, hidden))], None)],
                             [[0, 1]] * batch, q, lims=lims)
    same(cfg, dirty, clean)


@pytest.mark.parametrize("batch", [1, 9])
@pytest.mark.parametrize("dtype,d", STREAM)
def test_keys_hidden_from_some_rows(dtype, d, batch):
    """Own keys after a row's token, and linked rows past its own limit, hold
    infinities and NaN: the rows that do not see them keep their result."""
    rng = np.random.default_rng(d + 7)
    n = 130
    cfg = narrow(dtype, d, (64, 200), batch, (n,) * batch, (n,) * batch)
    q = normal(rng, batch * n, 6, d) * np.float32(cfg.q_std)
    chunks = [(normal(rng, 64, 2, d), normal(rng, 64, 2, d)),
              (normal(rng, 200, 2, d), normal(rng, 200, 2, d))]
    ks, vs = normal(rng, batch * n, 2, d), normal(rng, batch * n, 2, d)
    late = [r * n + t for r in range(batch) for t in range(100, n)]
    clean, dirty = run_calls(cfg, [(chunks, (ks, vs)), (chunks, (spoil(ks, late), spoil(vs, late)))],
                             [[0, 1]] * batch, q)
    see = np.arange(batch * n) % n < 100
    same(cfg, dirty, clean, see)
    # linked rows: the second chunk's rows 70.. are seen by every third row only
    lims = np.where(np.arange(batch * n) % 3 == 0, 264, 134).astype(np.int32)
    cross = narrow(dtype, d, (64, 200), batch, (n,) * batch, None)
    bad = (chunks[1][0], spoil(chunks[1][1], range(70, 200)))
    clean, dirty = run_calls(cross, [(chunks, None), ([chunks[0], bad], None)], [[0, 1]] * batch, q,
                             lims=lims)
    same(cfg, dirty, clean, lims == 134)


@pytest.mark.parametrize("batch", [1, 9])
@pytest.mark.parametrize("dtype,d", STREAM)
def test_visible_infinite_value(dtype, d, batch):
    """One infinite value seen by every row: its dim is infinite, the others
    keep their result."""
    rng = np.random.default_rng(d + 8)
    cfg = narrow(dtype, d, (64, 200), batch, (20,) * batch, (20,) * batch)
    q = normal(rng, batch * 20, 6, d) * np.float32(cfg.q_std)
    chunks = [(normal(rng, 64, 2, d), normal(rng, 64, 2, d)),
              (normal(rng, 200, 2, d), normal(rng, 200, 2, d))]
    own = (normal(rng, batch * 20, 2, d), normal(rng, batch * 20, 2, d))
    v = chunks[1][1].copy()
    v[33, :, 5] = math.inf
    clean, dirty = run_calls(cfg, [(chunks, own), ([chunks[0], (chunks[1][0], v)], own)],
                             [[0, 1]] * batch, q)
    assert (dirty[0][:, :, 5] == math.inf).all()
    rest = np.arange(d) != 5
    same(cfg, (dirty[0][:, :, rest], dirty[1]), (clean[0][:, :, rest], clean[1]))


@pytest.mark.parametrize("splits", [2, 3, 5, 6, 9, 21, 30])
def test_infinite_value_in_the_last_piece(splits):
    """Split counts that leave the combine's last group of pieces part empty: an
    infinite sum of the last piece stays infinite."""
    rng = np.random.default_rng(splits)
    cfg = narrow(W.BF16, 128, (640, 1300), 1, (2,), None, decode=True)
    q = normal(rng, 2, 6, 128) * np.float32(cfg.q_std)
    chunks = [(normal(rng, n, 2, 128), normal(rng, n, 2, 128)) for n in (640, 1300)]
    v = chunks[1][1].copy()
    v[1299, :, 5] = math.inf
    clean, dirty = run_calls(cfg, [(chunks, None), ([chunks[0], (chunks[1][0], v)], None)],
                             [[0, 1]], q, splits=splits)
    assert (dirty[0][:, :, 5] == math.inf).all()
    rest = np.arange(128) != 5
    assert np.array_equal(clean[0][:, :, rest], dirty[0][:, :, rest])


@pytest.mark.parametrize("own", [1, 5, 40])
def test_decode_last_own_value_infinite(own):
    """The decode kernel's in-place own tile reads past the last own key as that
    key again, masked: an infinite value of it stays infinite."""
    rng = np.random.default_rng(own)
    cfg = narrow(W.BF16, 128, (64, 200), 1, (1,), (own,), decode=True)
    q = normal(rng, 1, 6, 128) * np.float32(cfg.q_std)
    chunks = [(normal(rng, n, 2, 128), normal(rng, n, 2, 128)) for n in (64, 200)]
    ks, vs = normal(rng, own, 2, 128), normal(rng, own, 2, 128)
    bad = vs.copy()
    bad[own - 1, :, 5] = math.inf
    clean, dirty = run_calls(cfg, [(chunks, (ks, vs)), (chunks, (ks, bad))], [[0, 1]], q)
    assert (dirty[0][:, :, 5] == math.inf).all()
    rest = np.arange(128) != 5
    assert np.array_equal(clean[0][:, :, rest], dirty[0][:, :, rest])


NAN_FORMS = {
    # (config arguments, query tokens, splits (None: prefill), limits)
    "d128": (dict(d_k=128, n_q_heads=8, n_kv_heads=2), 40, None, False),
    "d128_limits": (dict(d_k=128, n_q_heads=8, n_kv_heads=2), 40, None, True),
    "decode_d128": (dict(d_k=128, n_q_heads=8, n_kv_heads=2), 1, 5, False),
    "mla": (MLA, 9, None, False),
    "stream_f32": (dict(d_k=64, dtype=W.F32, n_q_heads=6, n_kv_heads=2), 9, None, False),
    "stream_bf16": (dict(d_k=64, n_q_heads=6, n_kv_heads=2), 9, None, False),
    "stream_decode": (dict(d_k=64, n_q_heads=6, n_kv_heads=2), 2, 7, False),
    "small_decode": (dict(d_k=64, n_q_heads=6, n_kv_heads=2), 2, 7, False),
}


@pytest.mark.parametrize("every", [False, True])
@pytest.mark.parametrize("name", sorted(NAN_FORMS))
def test_nan_survives_a_split(name, every):
    """NaN keys that every row sees, in one piece of a split call or in every
    piece: the output rows are NaN, not the other pieces' result and not zero."""
    kw, q_len, splits, limited = NAN_FORMS[name]
    rng = np.random.default_rng(3)
    batch = 1 if name == "small_decode" else 9
    cfg = W.small_config("nan", chunk_lens=(640,) * 8, batch=batch, links=(0, 0),
                         q_len=(q_len,) * batch, self_len=None, decode=splits is not None, **kw)
    hkv, mla = cfg.n_kv_heads, cfg.kind == W.MLA
    q = normal(rng, batch * q_len, cfg.n_q_heads, cfg.d_k) * np.float32(cfg.q_std)
    chunks = []
    for i in range(8):
        k = normal(rng, 640, hkv, cfg.d_k)
        if every:
            k[::8] = math.nan
        elif i == 2:
            k[5] = math.nan
        chunks.append((k, None if mla else normal(rng, 640, hkv, cfg.d_v)))
    lims = None
    if limited:
        lims = (8 * 640 - np.arange(batch * q_len)).astype(np.int32)
    (out, _), = run_calls(cfg, [(chunks, None)], [list(range(8))] * batch, q, lims=lims,
                          splits=splits or 0)
    assert np.isnan(out).all()


@pytest.mark.parametrize("decode", [False, True])
@pytest.mark.parametrize("dtype,d", [(W.F32, 64), (W.F32, 128), (W.BF16, 32), (W.BF16, 64)])
def test_lse_rounded_once(dtype, d, decode):
    """The streaming kernel's log-sum-exp, unsplit and through the combine: its
    one rounding to fp32 is a relative 2^-24 / sqrt(3) = 3.4e-8 in the root mean
    square at most (the sum below it averages its roundings out); adding and
    scaling in log2 took three, 5.2e-8 to 5.6e-8."""
    q = (2,) * 9 if decode else (40,) * 9
    cfg = narrow(dtype, d, (700, 1300, 900), 9, q, None, decode=decode)
    links = [[0, 1, 2]] * 9
    wl = W.make_workload(cfg)
    chunks = [W.make_chunk(cfg, c) for c in range(3)]
    wide = (lambda x: x) if dtype == W.F32 else W.bf16_bits_to_f32
    for splits in ((1, 6) if decode else (0,)):
        (_, lse), = run_calls(cfg, [([(wide(k), wide(v)) for k, v in chunks], None)], links,
                              wide(wl.q), splits=splits)
        _, ref = ref_link(cfg, [[chunks[c] for c in l] for l in links], wl.q, wl.plan.q_offsets)
        assert np.linalg.norm(lse - ref) <= 4e-8 * np.linalg.norm(ref)
