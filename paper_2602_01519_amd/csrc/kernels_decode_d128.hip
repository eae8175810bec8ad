// bf16 GQA link attention for decode-shaped requests on gfx950, head dim 128.
//
// Decode reads every linked key once per query token (a generated token is a
// query token, Sec. 4), so the work is a stream over the request's
// concatenated chunk KV (Sec. 4.2) bounded by HBM bandwidth, not by math.
// Each wave owns one kv head of a work item (a piece of a request's keys) and streams its
// key range in 32-key tiles straight from HBM into registers, already in the
// operand layout of v_mfma_f32_16x16x32_bf16:
//   S^T[32 keys][16 cols] = K . Q^T    2 key blocks x 4 d steps  (8 MFMAs)
//   O^T[128][16 cols]    += V^T . P^T  8 value blocks x 1 step   (8 MFMAs)
// The 16 columns are the work item's rows (query token x GQA head, at most
// 16; unused columns are zero). The next tile's 16 x 16-byte loads per lane
// are in flight while the current tile is computed (register double
// buffering, loop unrolled by two), so each wave keeps 16 KB in flight.
//
// Row permutation: M index m of key block b reads key row 8*(m/4) + 4*b +
// m%4, so after QK^T lane l holds the scores of keys 8*(l/16) + 0..7 (four
// per block) for column l%16 -- exactly the 8 keys its PV operand needs, and
// the matching V^T operand is one 16-byte load of those 8 keys.
//
// Softmax: log2 domain, exact running max per tile (column max over the 4
// lane groups by two lane swaps), unnormalised partial (o, m, l) written per
// split and merged by the log-sum-exp combine (or normalised here when the
// range is not split).
#include "pic_internal.hpp"

namespace pic {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kD = 128;
constexpr int kT = 32;            // keys per decode tile
constexpr int kCols = 16;         // MFMA N: rows of a work item
constexpr int kWaves = 4;

__device__ __forceinline__ bf16x8 as_bf16x8(uint4 u) { return __builtin_bit_cast(bf16x8, u); }

// Reduction over the 4 lane groups (l, l^16, l^32, l^48) of a column.
__device__ __forceinline__ float col_max(float x) {
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float col_sum(float x) {
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// One tile's operands as loaded: K rows for the 2 key blocks x 4 d steps,
// V^T rows for the 8 value blocks.
struct Tile {
  uint4 k[8];
  uint4 v[8];
};

// Uniform facts of the tile being loaded / computed.
struct TileInfo {
  const char *k;    // first K row of the tile, kv head applied (bytes)
  const char *v;    // the tile's V^T panel, kv head applied
  int nvalid;       // valid keys in the tile
  int j0;           // key index of the tile's first key within its link
  int own;          // own-KV tile (causal mask)
};

struct Cursor {
  const_links links;       // the request's links, from the item's first on
  int li;                  // current link
  const char *k, *v;       // its K / V^T blocks
  int len, lp, tile0, end; // its tokens, padded tokens, first tile, tile after its last (32-key)
  int kvh;
  int doc_tiles32;         // 32-key tiles over the documents
};

__device__ __forceinline__ void cursor_set(Cursor &c, const void *k, const void *v, int len, int lp,
                                           int tile0) {
  c.k = (const char *)k;
  c.v = (const char *)v;
  c.len = len;
  c.lp = lp;
  c.tile0 = tile0 * (kTile / kT);
  c.end = c.tile0 + (len + kTile - 1) / kTile * (kTile / kT);
}

// Tile t (32-key units, t only grows) of the request.
__device__ __forceinline__ TileInfo tile_info(Cursor &c, int t) {
  while (t >= c.end) {
    ++c.li;
    cursor_set(c, c.links[c.li].k, c.links[c.li].v, c.links[c.li].len, c.links[c.li].lp,
               c.links[c.li].tile0);
  }
  const int tt = t - c.tile0;
  TileInfo r;
  r.nvalid = min(kT, c.len - tt * kT);
  r.j0 = tt * kT;
  r.own = 0;
  r.k = c.k + ((int64_t)c.kvh * c.lp + tt * kT) * kD * 2;
  r.v = c.v + ((int64_t)c.kvh * kD * c.lp + tt * kT * kD) * 2;   // the tile's V^T panel
  return r;
}

// Per-lane byte offsets of the tile's loads: K block b, step s: key row
// krow_b, d = 32 s + 8 (l/16); V block b: value row 16 b + l%16 of the
// tile's 32-key panel, keys 8 (l/16) .. +7 (two lanes of a 16-lane group
// read one 128-byte line).
// The keys are read once per call: the loads carry the nontemporal hint
// (streaming, measured 11% faster on a plain read stream).
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) const u32x4 *global_u32x4;
__device__ __forceinline__ uint4 load_nt(const char *p) {
  const u32x4 w = __builtin_nontemporal_load((global_u32x4)p);
  return make_uint4(w.x, w.y, w.z, w.w);
}

// Not live: the lanes of a load all read the same 16 bytes (one line), for
// the load that past the last tile only keeps the number of loads in flight
// fixed.
__device__ __forceinline__ void load_tile(const TileInfo &r, int lane, bool live, Tile &x) {
  const int grp = lane >> 4, m = lane & 15;
  const uint32_t mask = live ? ~0u : 0u;
  const uint32_t koff = (uint32_t)(((8 * (m >> 2) + (m & 3)) * kD + 8 * grp) * 2) & mask;
  const uint32_t voff = (uint32_t)(m * kT * 2 + 16 * grp) & mask;
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int s = 0; s < 4; ++s)
      x.k[b * 4 + s] = load_nt(r.k + koff + (4 * b * kD + 32 * s) * 2);
#pragma unroll
  for (int b = 0; b < 8; ++b) x.v[b] = load_nt(r.v + voff + 16 * b * kT * 2);
}

// Own-KV tile read in place: keys j0 .. of the request's token-major own rows
// (k, v: its first own row, kv head applied; stride: bytes per token). Keys
// past the last own one reread it: their scores are masked, and their values
// are zeros here, since the last key's would turn an infinite sum into NaN
// (0 x infinity). 2-byte gathers of the token-major values, once per kv head,
// beat a prologue that lays the own KV out at every length measured, step
// times, laid out -> in place: 64 requests over 16 links of 1024, 1 own token
// 603 -> 592 us, 128 618 -> 596, 1024 776 -> 616; 6 over 6 x 512, 1 to 128
// level, 1024 39.1 -> 29.5; 8 over 2 x 512, 16,384 271 -> 76.
__device__ __forceinline__ void load_own(const char *k, const char *v, int64_t stride, int j0,
                                         int last, int lane, Tile &x) {
  const int grp = lane >> 4, m = lane & 15;
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const char *row = k + min(j0 + 8 * (m >> 2) + 4 * b + (m & 3), last) * stride + 16 * grp;
#pragma unroll
    for (int s = 0; s < 4; ++s) x.k[b * 4 + s] = *(const uint4 *)(row + 64 * s);
  }
  uint32_t w[8][4];
#pragma unroll
  for (int b = 0; b < 8; ++b)
#pragma unroll
    for (int i = 0; i < 4; ++i) w[b][i] = 0;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int key = j0 + 8 * grp + i;
    const uint16_t *row = (const uint16_t *)(v + min(key, last) * stride) + m;
    const uint32_t keep = key <= last ? 0xffffu : 0u;
#pragma unroll
    for (int b = 0; b < 8; ++b) w[b][i >> 1] |= (row[16 * b] & keep) << (16 * (i & 1));
  }
#pragma unroll
  for (int b = 0; b < 8; ++b) x.v[b] = make_uint4(w[b][0], w[b][1], w[b][2], w[b][3]);
}

struct State {
  f32x4 o[8];       // O^T blocks: value rows 16 b + 4 (l/16) + i, column l%16
  float m, l;       // running max (log2 domain, per column) and this lane's partial sum
};

__device__ __forceinline__ void compute_tile(const Tile &x, const TileInfo &r,
                                             const bf16x8 (&qf)[4], State &st, int lane,
                                             int lim, float sc) {
  f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    s0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(x.k[s]), qf[s], s0, 0, 0, 0);
    s1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(x.k[4 + s]), qf[s], s1, 0, 0, 0);
  }
  // s0[i]: key 8 (l/16) + i, s1[i]: key 8 (l/16) + 4 + i, column l%16
  const int kbase = 8 * (lane >> 4);
  if (r.own || r.nvalid < kT) {
    const int kl = (r.own ? min(lim - r.j0, r.nvalid - 1) : r.nvalid - 1) - kbase;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (i > kl) s0[i] = -INFINITY;
      if (4 + i > kl) s1[i] = -INFINITY;
    }
  }
  float tmax = fmaxf(fmaxf(fmaxf(s0[0], s0[1]), fmaxf(s0[2], s0[3])),
                     fmaxf(fmaxf(s1[0], s1[1]), fmaxf(s1[2], s1[3])));
  tmax = col_max(tmax);
  const float mnew = fmaxf(st.m, tmax * sc);
  if (mnew > st.m) {             // per lane: rescale this column's state
    const float alpha = __builtin_amdgcn_exp2f(st.m - mnew);   // 0 when st.m = -inf
    st.l *= alpha;
#pragma unroll
    for (int b = 0; b < 8; ++b) st.o[b] *= alpha;
    st.m = mnew;
  }
  const float neg_m = st.m == -INFINITY ? 0.f : -st.m;
  bf16x8 pf;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    pf[i] = (__bf16)__builtin_amdgcn_exp2f(__builtin_fmaf(s0[i], sc, neg_m));
    pf[4 + i] = (__bf16)__builtin_amdgcn_exp2f(__builtin_fmaf(s1[i], sc, neg_m));
  }
  const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
#pragma unroll
  for (int i = 0; i < 8; i += 2) {
    const bf16x2 pp = {pf[i], pf[i + 1]};
    st.l = __builtin_amdgcn_fdot2_f32_bf16(pp, ones, st.l, false);
  }
#pragma unroll
  for (int b = 0; b < 8; ++b)
    st.o[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(x.v[b]), pf, st.o[b], 0, 0, 0);
}

__global__ __launch_bounds__(256, 2) void link_decode_d128_kernel(LinkParams p) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // one (item, kv head) per wave
  const int u = blockIdx.x * kWaves + wave;
  if (u >= p.n_items * p.n_kv_heads) return;
  const int kvh = u % p.n_kv_heads;
  const WorkItem it = load_item(p.items, u / p.n_kv_heads);
  const ReqEntry R = item_request(it);
  const int group = p.group;
  const int nrows = R.lq * group;                 // <= kCols (checked by the planner)
  const int t_begin = it.t_begin, t_end = it.t_end;

  Cursor cur;
  cur.links = (const_links)p.links + it.link;
  cur.li = 0;
  cur.kvh = kvh;
  cur.doc_tiles32 = R.doc_tiles * (kTile / kT);
  cursor_set(cur, it.k, it.v, it.len, it.lp, it.tile0);

  // This lane's column (row of the work item).
  const int col = lane & 15;
  const bool cvalid = col < nrows;
  const int qi = cvalid ? col / group : 0;
  const int qh = kvh * group + (cvalid ? col % group : 0);
  const int lim = cvalid ? qi + R.ls - R.lq : -1;
  const int64_t orow = (int64_t)(R.q0 + qi) * p.n_q_heads + qh;

  // Own KV in place: its tiles come first (the order of the keys does not
  // matter to the sums), while the first document tile is in flight.
  const int doc_end = min(t_end, cur.doc_tiles32);
  Tile ta, tb;
  TileInfo ia{}, ib{};
  if (t_begin < doc_end) {
    ia = tile_info(cur, t_begin);
    load_tile(ia, lane, true, ta);
  }
  // Q operand: Q^T[d = 32 s + 8 (l/16) + 0..7][col]
  bf16x8 qf[4];
  {
    const uint4 *qrow = (const uint4 *)((const uint16_t *)p.q + orow * kD);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      uint4 v = make_uint4(0, 0, 0, 0);
      if (cvalid) v = qrow[4 * s + (lane >> 4)];
      qf[s] = as_bf16x8(v);
    }
  }
  State st;
#pragma unroll
  for (int b = 0; b < 8; ++b) st.o[b] = f32x4{0.f, 0.f, 0.f, 0.f};
  st.m = -INFINITY;
  st.l = 0.f;
  const float sc = p.scale_log2;

  if (t_end > cur.doc_tiles32) {
    const int64_t at = ((int64_t)it.tok0 * p.n_kv_heads + kvh) * kD * 2;
    const int64_t stride = (int64_t)p.n_kv_heads * kD * 2;
    const int own_end = min(t_end, cur.doc_tiles32 + (R.ls + kT - 1) / kT);
    for (int t = max(t_begin, cur.doc_tiles32); t < own_end; ++t) {
      ib.own = 1;
      ib.j0 = (t - cur.doc_tiles32) * kT;
      ib.nvalid = min(kT, R.ls - ib.j0);
      load_own((const char *)p.k_self + at, (const char *)p.v_self + at, stride, ib.j0, R.ls - 1,
               lane, tb);
      compute_tile(tb, ib, qf, st, lane, lim, sc);
    }
  }
  // The loads past the last tile read next to nothing of it: a branch around
  // them makes the compiler wait for every load in flight where the paths
  // meet, so that no load ran under the arithmetic of its own wave (64
  // requests x 16 links of 1024: 670 -> 660 us).
  for (int t = t_begin; t < doc_end; t += 2) {
    ib = tile_info(cur, min(t + 1, doc_end - 1));
    load_tile(ib, lane, t + 1 < doc_end, tb);
    compute_tile(ta, ia, qf, st, lane, lim, sc);
    if (t + 1 >= doc_end) break;
    ia = tile_info(cur, min(t + 2, doc_end - 1));
    load_tile(ia, lane, t + 2 < doc_end, ta);
    compute_tile(tb, ib, qf, st, lane, lim, sc);
  }

  const float ltot = col_sum(st.l);
  if (!cvalid) return;
  // lane l holds value rows 16 b + 4 (l/16) + i of column l%16
  const int r4 = 4 * (lane >> 4);
  if (it.part < 0) {
    const float inv = ltot > 0.f ? 1.f / ltot : 0.f;
    uint16_t *out = (uint16_t *)p.out + orow * kD;
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      __bf16 v4[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) v4[i] = (__bf16)(st.o[b][i] * inv);
      *(uint2 *)(out + 16 * b + r4) = __builtin_bit_cast(uint2, v4);
    }
    if (p.lse && lane < 16)
      p.lse[orow] = ltot > 0.f ? (st.m + log2f(ltot)) * 0.69314718055994531f : -INFINITY;
  } else {
    const int64_t prow = it.part + (orow - (int64_t)R.q0 * p.n_q_heads);
    float *po = p.part_o + prow * kD;
#pragma unroll
    for (int b = 0; b < 8; ++b)
      *(float4 *)(po + 16 * b + r4) = make_float4(st.o[b][0], st.o[b][1], st.o[b][2], st.o[b][3]);
    if (lane < 16) {
      p.part_m[prow] = partial_max(st.m, ltot);
      p.part_l[prow] = ltot;
    }
  }
}

}  // namespace

int decode_d128_max_rows() { return kCols; }

hipError_t launch_link_decode_d128(const LinkParams &p, hipStream_t st, const char **name) {
  *name = "link_decode_d128_kernel";
  const int64_t items = (int64_t)p.n_items * p.n_kv_heads;
  dim3 grid((unsigned)((items + kWaves - 1) / kWaves));
  hipLaunchKernelGGL(link_decode_d128_kernel, grid, dim3(64 * kWaves), 0, st, p);
  return hipGetLastError();
}

}  // namespace pic
