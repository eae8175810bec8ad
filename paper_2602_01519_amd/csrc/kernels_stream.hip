// GQA link attention on gfx950 matrix cores for fp32 caches and for bf16
// caches with narrow heads (d_k = d_v = D): prefill- and decode-shaped calls.
//
// Every wave streams its own key range: 32-key tiles go from memory straight
// into registers in the operand layout of the 16x16 matrix instructions, the
// next tile's loads in flight under the current tile's arithmetic, with no
// LDS staging and no barrier in the loop. Keys are walked as in the other
// kernels: linked chunks in link order (Sec. 4.2: concatenated, no mask),
// then the request's own KV (Sec. 4.1: causal, bottom-right aligned).
//
// A wave holds CB column blocks of 16 rows (a row is a query token and a
// query head of the GQA group), so every K and V register feeds CB matrix
// instructions. Per tile:
//   S^T[32 keys][16 rows] = K Q^T        per column block
//   softmax against a running max that only moves when a score passes it by
//   2^64 (fp32 keeps its relative precision at any such magnitude)
//   O^T[D][16 rows] += V^T P^T
// A wave whose sums come out beyond 2^115, infinite or NaN takes its rows
// again on the vector ALU (rows_alone), but for rows whose probabilities sum
// to NaN, which stay NaN in any order. There the max follows every key, so
// probabilities stay at or below one and sums overflow only where the values'
// own sums do, and a key that a row does not see adds nothing to it whatever
// it holds (0 x infinity is NaN). Other calls pay half a maximum per
// sum at the end of a piece: 8 ragged bf16 requests of 30..300 tokens 148.1 ->
// 148.6 us, 12 fp32 ones of 20..130 tokens 65.1 -> 65.3 (a max that follows
// every tile instead: 176 and 67.1).
// The scores a lane receives are the keys its operand of the value product
// needs, so probabilities never leave its registers:
//   fp32 (v_mfma_f32_16x16x4_f32): A lane l = (row l % 16, k-slot l / 16);
//     contraction step (j, i) takes head dims 16 j + 4 (l / 16) + i, so a
//     lane's operands are whole 16-byte loads; score register i of key block
//     b is key 16 b + 4 (l / 16) + i.
//   bf16 (v_mfma_f32_16x16x32_bf16): key block b's M index m reads key row
//     8 (m / 4) + 4 b + m % 4, so the registers of both blocks are keys
//     8 (l / 16) + 0 .. 7.
// The probabilities stay fp32. For bf16 caches the value product takes them
// as the sum of two bf16 numbers (p = hi + lo, |p - hi - lo| <= 2^-17 p, far
// below the rounding of the bf16 output), two matrix instructions per value
// block; row sums add the fp32 probabilities.
//
// Work mapping: a workgroup's four waves are 4 / kpar row blocks times kpar
// parts of one key range. Calls with many rows take kpar = 1: the four waves
// walk the same tiles, which one of them brings into the CU's cache. Calls
// with few rows split the keys over the waves too and merge the (m, l, O) of
// the parts through LDS at the end.
//
// What bounds it (counters of the two ragged batches above): a wave's own
// chain of instructions, since such batches keep 0.95 waves per SIMD. bf16 at
// D = 64: 41 cycles of vector issue per score and lane (exponential, sum, the
// hi / lo split; 6 of them the matrix instructions' issue) and 24 matrix
// cycles; the vector ALU issues in 42% of the SIMD cycles, the matrix cores are
// busy in 25%. fp32: matrix cores 41%, vector ALU 11%, and two thirds of the
// wave cycles wait for a matrix instruction before the next. Measured figures
// stand at launch_link_stream.
#include "pic_internal.hpp"

#include <cstddef>
#include <type_traits>

namespace pic {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

constexpr int kT = 32;            // keys per tile
constexpr int kWaves = 4;
constexpr float kJump = 64.0f;    // log2: the running max moves past it
// Sums up to this size stay finite when the parts of a workgroup and the
// pieces of a request (at most 4 x 256) are added up.
constexpr float kSafeSum = 0x1p115f;

__device__ __forceinline__ int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ bf16x8 as_bf16x8(uint4 u) { return __builtin_bit_cast(bf16x8, u); }

// Reductions over the 4 lane groups (l, l ^ 16, l ^ 32, l ^ 48) of a row.
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

template <typename T, int D>
struct Shape {
  static constexpr bool F32 = sizeof(T) == 4;
  static constexpr int E = 16 / (int)sizeof(T);          // elements per 16-byte unit
  static constexpr int KU = D * (int)sizeof(T) / 64;     // 16-byte units per lane and key row
  static constexpr int NB = D / 16;                      // value blocks
  static constexpr int VU = F32 ? 2 : 1;                 // 16-byte units per lane and value block
};

// One tile's operands as loaded: K units [key block][unit], V^T units
// [value block][unit].
template <typename T, int D>
struct Tile {
  uint4 k[2][Shape<T, D>::KU];
  uint4 v[Shape<T, D>::NB][Shape<T, D>::VU];
};

// Uniform facts of a tile.
struct TileInfo {
  const char *k;    // first K row of the tile, kv head applied (bytes)
  const char *v;    // the tile's V^T panel, kv head applied
  int nvalid;       // valid keys in the tile (0 or less: none)
  int j0;           // key index of the tile's first key within its link
  int tok;          // ... within the request's linked rows (document tiles)
  int own;          // own-KV tile (causal mask)
};

// Link and request tables are read through the constant address space: the
// cursor over the links lives in scalar registers.
typedef __attribute__((address_space(4))) const ReqEntry *const_reqs;
typedef __attribute__((address_space(4))) const int32_t *const_ints;

struct Cursor {
  const_links links;
  int li;
  const char *k, *v;
  int len, lp, tile0, end, tok0;   // tile0, end: in 32-key tiles
  int kvh, doc_tiles;              // doc_tiles: in 32-key tiles
};

__device__ __forceinline__ void cursor_set(Cursor &c, const void *k, const void *v, int len, int lp,
                                           int tile0, int tok0) {
  c.k = (const char *)k;
  c.v = (const char *)v;
  c.len = len;
  c.lp = lp;
  c.tile0 = tile0 * (kTile / kT);
  c.tok0 = tok0;
  c.end = c.tile0 + (len + kTile - 1) / kTile * (kTile / kT);
}
__device__ __forceinline__ void cursor_load(Cursor &c) {
  cursor_set(c, c.links[c.li].k, c.links[c.li].v, c.links[c.li].len, c.links[c.li].lp,
             c.links[c.li].tile0, c.links[c.li].tok0);
}

// The link of a small call's request that holds its 64-key tile t: the lanes
// read the first tiles of all its links at once (kSmallLinks <= 64).
__device__ __forceinline__ int seek_link(const_links links, int nlinks, int t, int lane) {
  const bool before = lane < nlinks && links[min(lane, nlinks - 1)].tile0 <= t;
  return uni(max(0, __popcll(__ballot(before)) - 1));
}

// Tile t of the request (t only grows).
template <typename T, int D>
__device__ __forceinline__ TileInfo tile_info(Cursor &c, int t) {
  while (t >= c.end) {
    ++c.li;
    cursor_load(c);
  }
  const int tt = t - c.tile0;
  TileInfo r;
  r.nvalid = min(kT, c.len - tt * kT);
  r.j0 = tt * kT;
  r.tok = c.tok0 + tt * kT;
  r.own = t >= c.doc_tiles;
  r.k = c.k + ((int64_t)c.kvh * c.lp + tt * kT) * (D * (int)sizeof(T));
  r.v = c.v + ((int64_t)c.kvh * c.lp + tt * kT) * (D * (int)sizeof(T));   // a panel is kT x D too
  return r;
}

// koff / voff: this lane's byte offsets within a tile's K rows and panel.
template <typename T, int D>
__device__ __forceinline__ void load_tile(const TileInfo &r, uint32_t koff, uint32_t voff,
                                          Tile<T, D> &x) {
  using S = Shape<T, D>;
  constexpr int kRowBlock = (S::F32 ? 16 : 4) * D * (int)sizeof(T);   // key block 1 after block 0
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int j = 0; j < S::KU; ++j)
      x.k[b][j] = *(const uint4 *)(r.k + koff + b * kRowBlock + j * 64);
#pragma unroll
  for (int b = 0; b < S::NB; ++b)
#pragma unroll
    for (int u = 0; u < S::VU; ++u)
      x.v[b][u] = *(const uint4 *)(r.v + voff + b * 16 * kT * (int)sizeof(T) + u * 64);
}

// Own-KV tiles of a small call, read in place: keys j0 .. of the request's
// token-major rows (k, v: its first own row, kv head applied; stride: bytes
// per token). Keys past the last own one reread it; they are masked.
struct OwnRows {
  const char *k, *v;
  int64_t stride;
  int last;
};
template <typename T, int D>
__device__ __forceinline__ void load_own(const OwnRows &o, int j0, int lr, int lg,
                                         Tile<T, D> &x) {
  using S = Shape<T, D>;
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const int key = S::F32 ? 16 * b + lr : 8 * (lr >> 2) + 4 * b + (lr & 3);
    const char *row = o.k + min(j0 + key, o.last) * o.stride + 16 * lg;
#pragma unroll
    for (int j = 0; j < S::KU; ++j) x.k[b][j] = *(const uint4 *)(row + j * 64);
  }
#pragma unroll
  for (int u = 0; u < S::VU; ++u) {
    // the unit's keys: 16 u + 4 lg + 0..3 (fp32), 8 lg + 0..7 (bf16)
    uint32_t w[S::NB][4];
#pragma unroll
    for (int b = 0; b < S::NB; ++b)
#pragma unroll
      for (int i = 0; i < 4; ++i) w[b][i] = 0;
#pragma unroll
    for (int i = 0; i < S::E; ++i) {
      const int key = S::F32 ? 16 * u + 4 * lg + i : 8 * lg + i;
      const T *row = (const T *)(o.v + min(j0 + key, o.last) * o.stride) + lr;
#pragma unroll
      for (int b = 0; b < S::NB; ++b) {
        if constexpr (S::F32)
          w[b][i] = __float_as_uint(row[16 * b]);
        else
          w[b][i >> 1] |= (uint32_t)row[16 * b] << (16 * (i & 1));
      }
    }
#pragma unroll
    for (int b = 0; b < S::NB; ++b) x.v[b][u] = make_uint4(w[b][0], w[b][1], w[b][2], w[b][3]);
  }
}

__device__ __forceinline__ float unit(const uint4 &u, int i) {
  return __uint_as_float(i == 0 ? u.x : i == 1 ? u.y : i == 2 ? u.z : u.w);
}

template <typename T, int D, int CB>
struct State {
  f32x4 o[CB][Shape<T, D>::NB];   // O^T: value dims 16 b + 4 (l / 16) + i, row l % 16
  float m[CB], l[CB];             // running max (log2 domain), this lane's partial row sum
};

template <typename T, int D, int CB>
__device__ __forceinline__ void compute_tile(const Tile<T, D> &x, const TileInfo &r,
                                             const uint4 (&qf)[CB][Shape<T, D>::KU],
                                             State<T, D, CB> &st, int lg, const int (&lim)[CB],
                                             const int (&dl)[CB], int wmin, float sc) {
  using S = Shape<T, D>;
  f32x4 s[CB][2];
#pragma unroll
  for (int c = 0; c < CB; ++c)
#pragma unroll
    for (int b = 0; b < 2; ++b) s[c][b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < S::KU; ++j) {
    if constexpr (S::F32) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int c = 0; c < CB; ++c)
            s[c][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(unit(x.k[b][j], i), unit(qf[c][j], i),
                                                           s[c][b], 0, 0, 0);
    } else {
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int c = 0; c < CB; ++c)
          s[c][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
              as_bf16x8(x.k[b][j]), as_bf16x8(qf[c][j]), s[c][b], 0, 0, 0);
    }
  }
  // key of score register i of block b, less the lane's own part of it
  auto key = [](int b, int i) { return S::F32 ? 16 * b + i : 4 * b + i; };
  const int kbase = (S::F32 ? 4 : 8) * lg;
  if (r.own || r.nvalid < kT || r.tok + kT > wmin) {
#pragma unroll
    for (int c = 0; c < CB; ++c) {
      const int kl = (r.own ? min(lim[c] - r.j0, r.nvalid - 1) : min(dl[c] - r.tok, r.nvalid) - 1) -
                     kbase;
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (key(b, i) > kl) s[c][b][i] = -INFINITY;
    }
  }
  // The running max moves only if some score of the wave passes it by
  // 2^64 (or a row with a visible key has none yet).
  float tmax[CB];
  bool jump = false;
#pragma unroll
  for (int c = 0; c < CB; ++c) {
    tmax[c] = fmaxf(fmaxf(fmaxf(s[c][0][0], s[c][0][1]), fmaxf(s[c][0][2], s[c][0][3])),
                    fmaxf(fmaxf(s[c][1][0], s[c][1][1]), fmaxf(s[c][1][2], s[c][1][3])));
    jump |= !(__builtin_fmaf(tmax[c], sc, -st.m[c]) <= kJump) && tmax[c] != -INFINITY;
  }
  if (__builtin_expect(__any(jump), 0)) {
#pragma unroll
    for (int c = 0; c < CB; ++c) {
      const float mnew = fmaxf(st.m[c], col_max(tmax[c]) * sc);
      const float alpha = mnew == st.m[c] ? 1.f : __builtin_amdgcn_exp2f(st.m[c] - mnew);
      st.m[c] = mnew;
      st.l[c] *= alpha;
#pragma unroll
      for (int b = 0; b < S::NB; ++b) st.o[c][b] *= alpha;
    }
  }
#pragma unroll
  for (int c = 0; c < CB; ++c) {
    const float neg_m = st.m[c] == -INFINITY ? 0.f : -st.m[c];
    float p[2][4];
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        p[b][i] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[c][b][i], sc, neg_m));
    st.l[c] += ((p[0][0] + p[0][1]) + (p[0][2] + p[0][3])) +
               ((p[1][0] + p[1][1]) + (p[1][2] + p[1][3]));
    if constexpr (S::F32) {
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int b = 0; b < S::NB; ++b)
            st.o[c][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(unit(x.v[b][u], i), p[u][i],
                                                              st.o[c][b], 0, 0, 0);
    } else {
      // hi: p rounded to bf16; lo: the rest, p - hi (one dot product each:
      // bf16 products are exact), rounded to bf16
      bf16x8 hi, lo;
      // (-1, 0) and (0, -1), kept in scalar registers: the compiler writes
      // (-1, 0) as the inline constant -1.0, which the instruction reads as
      // the fp32 pattern, that is (0, -1)
      uint32_t c0 = 0x0000bf80u, c1 = 0xbf800000u;
      asm("" : "+s"(c0), "+s"(c1));
      const bf16x2 first = __builtin_bit_cast(bf16x2, c0), second = __builtin_bit_cast(bf16x2, c1);
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int i = 0; i < 4; i += 2) {
          const bf16x2 h = __builtin_convertvector((f32x2){p[b][i], p[b][i + 1]}, bf16x2);
          const f32x2 rest = {__builtin_amdgcn_fdot2_f32_bf16(h, first, p[b][i], false),
                              __builtin_amdgcn_fdot2_f32_bf16(h, second, p[b][i + 1], false)};
          const bf16x2 l = __builtin_convertvector(rest, bf16x2);
          hi[4 * b + i] = h[0];
          hi[4 * b + i + 1] = h[1];
          lo[4 * b + i] = l[0];
          lo[4 * b + i + 1] = l[1];
        }
#pragma unroll
      for (int b = 0; b < S::NB; ++b) {
        st.o[c][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(x.v[b][0]), hi, st.o[c][b],
                                                             0, 0, 0);
        st.o[c][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(x.v[b][0]), lo, st.o[c][b],
                                                             0, 0, 0);
      }
    }
  }
}

template <typename T>
__device__ __forceinline__ void store4(T *out, float a, float b, float c, float d);
template <>
__device__ __forceinline__ void store4<float>(float *out, float a, float b, float c, float d) {
  *(float4 *)out = make_float4(a, b, c, d);
}
template <>
__device__ __forceinline__ void store4<uint16_t>(uint16_t *out, float a, float b, float c,
                                                 float d) {
  const __bf16 v[4] = {(__bf16)a, (__bf16)b, (__bf16)c, (__bf16)d};
  *(uint2 *)out = __builtin_bit_cast(uint2, v);
}

// Element i of a 16-byte unit.
template <typename T>
__device__ __forceinline__ float element(const uint4 &u, int i) {
  if constexpr (sizeof(T) == 4) return unit(u, i);
  const uint32_t w = i < 2 ? u.x : i < 4 ? u.y : i < 6 ? u.z : u.w;
  return __uint_as_float(i & 1 ? w & 0xffff0000u : w << 16);
}

// A workgroup's piece of work and a wave's part of it.
struct Piece {
  ReqEntry R;
  Cursor cur;            // at the first tile (if there is one)
  int part_row;          // first partial row of the piece, -1: not split
  int nrows, wg_row0, row0;
  int t_begin, t_end;    // the wave's tiles
};

// kSmall: a small call, whose tables are kernel arguments and whose own-KV
// tiles are read in place (no prologue kernel before it). False: no such
// piece. kR: rows per wave.
template <bool kSmall, int kR>
__device__ __forceinline__ bool piece_of(const LinkParams &p, const_links links, const_reqs reqs,
                                         const_ints order, int block, int wave, int lane,
                                         Piece &w) {
  const int units = p.n_kv_heads * (kSmall ? p.batch * p.num_splits : p.n_items);
  const UnitBlock ub = unit_of_block(block, p.nrb, p.n_xcd, p.spread, units);
  if (ub.u >= units) return false;
  int p_begin = 0, p_end = 0;   // the piece, in 32-key tiles
  ReqEntry &R = w.R;
  Cursor &cur = w.cur;
  w.part_row = -1;
  if constexpr (kSmall) {
    const int grp = ub.u / p.num_splits, split = ub.u % p.num_splits;
    cur.kvh = grp % p.n_kv_heads;
    const_reqs rq = reqs + order[grp / p.n_kv_heads];
    R.link0 = rq->link0;
    R.nlinks = rq->nlinks;
    R.q0 = rq->q0;
    R.lq = rq->lq;
    R.s0 = rq->s0;
    R.ls = rq->ls;
    R.doc_tiles = rq->doc_tiles;
    R.tiles = rq->tiles;
    p_begin = (int)((int64_t)2 * R.tiles * split / p.num_splits);
    p_end = (int)((int64_t)2 * R.tiles * (split + 1) / p.num_splits);
    if (p.num_splits > 1) w.part_row = (split * p.total_q + R.q0) * p.n_q_heads;
    cur.links = links + R.link0;
  } else {
    const WorkItem it = load_item(p.items, ub.u / p.n_kv_heads);
    cur.kvh = ub.u % p.n_kv_heads;
    R = item_request(it);
    p_begin = it.t_begin;
    p_end = it.t_end;
    w.part_row = it.part;
    cur.links = links + it.link;
    cur.li = 0;
    cursor_set(cur, it.k, it.v, it.len, it.lp, it.tile0, it.tok0);
  }
  cur.doc_tiles = 2 * R.doc_tiles;
  const int kpar = p.kpar;
  w.nrows = R.lq * p.group;
  w.wg_row0 = ub.rb * (kWaves / kpar) * kR;
  if (w.wg_row0 >= w.nrows) return false;
  w.row0 = w.wg_row0 + (wave / kpar) * kR;

  // the piece's tiles up to the last own key the wave's last row sees, cut
  // into kpar parts
  w.t_begin = w.t_end = 0;
  if (w.row0 < w.nrows) {
    const int own_last = min(w.nrows - 1, w.row0 + kR - 1) / p.group + R.ls - R.lq;
    const int vis = own_last >= 0 ? min(2 * R.tiles, 2 * R.doc_tiles + own_last / kT + 1)
                                  : 2 * R.doc_tiles;
    const int n = max(0, min(p_end, vis) - p_begin), part = wave % kpar;
    w.t_begin = p_begin + n * part / kpar;
    w.t_end = p_begin + n * (part + 1) / kpar;
  }
  if constexpr (kSmall)
    if (w.t_begin < w.t_end) {
      cur.li = seek_link(cur.links, R.nlinks, w.t_begin / (kTile / kT), lane);
      cursor_load(cur);
    }
  return true;
}

// The own rows of a small call's request, for one kv head.
template <typename T, int D>
__device__ __forceinline__ OwnRows own_rows(const LinkParams &p, const ReqEntry &R, int kvh) {
  OwnRows own{};
  if (R.ls > 0) {
    const int64_t at = ((int64_t)R.s0 * p.n_kv_heads + kvh) * D * (int)sizeof(T);
    own.k = (const char *)p.k_self + at;
    own.v = (const char *)p.v_self + at;
    own.stride = (int64_t)p.n_kv_heads * D * sizeof(T);
    own.last = R.ls - 1;
  }
  return own;
}

// A wave's rows over its tiles, four at a time: (m, l, O) of row i to sm[i],
// sl[i], so[i * stride + dim]. Lane l takes key l % 32 of a tile and half of its
// head dims for the scores, value dims l and l + 64 for the sums, to which a
// row's hidden keys add zero. Four rows share each 16-byte load of keys and
// values: a call of 8 x 128 tokens over 8 x 512 rows, 32 heads on 8, all of
// whose rows come here takes 2.5 ms (bf16, 64 wide; one row at a time with
// element-wide loads 20, the vector-ALU kernel of the other shapes 1.6), where
// the matrix instructions take 0.08.
template <typename T, int D, bool kSmall>
__device__ __forceinline__ void rows_alone(const LinkParams &p, const Piece &w, int rows,
                                           int lane, float *so, int stride, float *sm,
                                           float *sl) {
  constexpr int kG = 4, E = Shape<T, D>::E, kUnits = D / 2 / E, kDims = D > 64 ? 2 : 1;
  const ReqEntry &R = w.R;
  const OwnRows own = own_rows<T, D>(p, R, w.cur.kvh);
  const int key = lane & 31, half = (lane >> 5) * (D / 2);
  const int dim = D < 64 ? lane % D : lane;
  const int n = min(rows, w.nrows - w.row0);
#pragma unroll 1
  for (int i0 = 0; i0 < n; i0 += kG) {
    const T *q[kG];
    int lim[kG], dl[kG];
    float m[kG], l[kG], o[kG][kDims];
#pragma unroll
    for (int g = 0; g < kG; ++g) {
      const int row = w.row0 + min(i0 + g, n - 1), qi = row / p.group;
      const int qh = w.cur.kvh * p.group + row % p.group;
      q[g] = (const T *)p.q + ((int64_t)(R.q0 + qi) * p.n_q_heads + qh) * D + half;
      lim[g] = qi + R.ls - R.lq;
      dl[g] = p.doc_lim ? p.doc_lim[R.q0 + qi] : kNoLimit;
      m[g] = -INFINITY;
      l[g] = 0.f;
#pragma unroll
      for (int j = 0; j < kDims; ++j) o[g][j] = 0.f;
    }
    Cursor cur = w.cur;
#pragma unroll 1
    for (int t = w.t_begin; t < w.t_end; ++t) {
      const TileInfo x = tile_info<T, D>(cur, t);
      int last[kG], most = -1;
#pragma unroll
      for (int g = 0; g < kG; ++g) {
        last[g] = x.own ? min(lim[g] - x.j0, x.nvalid - 1) : min(dl[g] - x.tok, x.nvalid) - 1;
        most = max(most, last[g]);
      }
      if (most < 0) continue;
      const bool place = kSmall && x.own;
      const T *k = place ? (const T *)(own.k + min(x.j0 + key, own.last) * own.stride)
                         : (const T *)x.k + key * D;
      float s[kG], pr[kG];
#pragma unroll
      for (int g = 0; g < kG; ++g) s[g] = 0.f;
#pragma unroll 2
      for (int u = 0; u < kUnits; ++u) {
        const uint4 ku = *(const uint4 *)(k + half + u * E);
#pragma unroll
        for (int g = 0; g < kG; ++g) {
          const uint4 qu = *(const uint4 *)(q[g] + u * E);
#pragma unroll
          for (int e = 0; e < E; ++e) s[g] += element<T>(qu, e) * element<T>(ku, e);
        }
      }
#pragma unroll
      for (int g = 0; g < kG; ++g) {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(s[g]),
                                                        __float_as_uint(s[g]), false, false);
        s[g] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
        s[g] = key <= last[g] ? s[g] * p.scale_log2 : -INFINITY;
        const float mnew = fmaxf(m[g], wave_max(s[g]));
        const float base = mnew == -INFINITY ? 0.f : mnew;
        pr[g] = key <= last[g] ? exp2f(s[g] - base) : 0.f;
        const float alpha = exp2f(m[g] - base);
        l[g] = l[g] * alpha + 0.5f * wave_sum(pr[g]);     // both halves hold the keys
        m[g] = mnew;
#pragma unroll
        for (int j = 0; j < kDims; ++j) o[g][j] *= alpha;
      }
#pragma unroll
      for (int j = 0; j < kDims; ++j) {
        const int e = dim + 64 * j;
        float v[kT];
        if (place) {
#pragma unroll
          for (int kk = 0; kk < kT; ++kk) {
            const T t1 = *((const T *)(own.v + min(x.j0 + kk, own.last) * own.stride) + e);
            v[kk] = sizeof(T) == 4 ? (float)t1 : __uint_as_float((uint32_t)t1 << 16);
          }
        } else {
#pragma unroll
          for (int u = 0; u < kT / E; ++u) {
            const uint4 vu = *(const uint4 *)((const T *)x.v + e * kT + u * E);
#pragma unroll
            for (int b = 0; b < E; ++b) v[u * E + b] = element<T>(vu, b);
          }
        }
#pragma unroll
        for (int kk = 0; kk < kT; ++kk)
#pragma unroll
          for (int g = 0; g < kG; ++g) {
            const float pk = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(pr[g]), kk));
            o[g][j] += pk * (kk <= last[g] ? v[kk] : 0.f);
          }
      }
    }
#pragma unroll
    for (int g = 0; g < kG; ++g) {
      if (i0 + g >= n) break;
      if (D >= 64 || lane < D)
#pragma unroll
        for (int j = 0; j < kDims; ++j) so[(i0 + g) * stride + dim + 64 * j] = o[g][j];
      if (lane == 0) {
        sm[i0 + g] = partial_max(m[g], l[g]);
        sl[i0 + g] = l[g];
      }
    }
  }
}

template <typename T, int D, int CB, bool kSmall>
__device__ __forceinline__ void stream_body(const LinkParams &p, const_links links,
                                            const_reqs reqs, const_ints order) {
  using S = Shape<T, D>;
  constexpr int kR = 16 * CB;              // rows per wave
  constexpr int kOS = D + 4;               // merge buffer row stride (floats)
  __shared__ __attribute__((aligned(16))) float so[kWaves][kR * kOS];
  __shared__ float sm[kWaves][kR], sl[kWaves][kR];

  const int lane = threadIdx.x & 63;
  const int wave = uni(threadIdx.x >> 6);
  const int lr = lane & 15, lg = lane >> 4;

  Piece w;
  if (!piece_of<kSmall, kR>(p, links, reqs, order, blockIdx.x, wave, lane, w)) return;
  const ReqEntry &R = w.R;
  Cursor &cur = w.cur;
  const int group = p.group, kpar = p.kpar, kvh = cur.kvh, part_row = w.part_row;
  const int nrows = w.nrows, wg_row0 = w.wg_row0, row0 = w.row0;
  const int t_begin = w.t_begin, t_end = w.t_end;

  int lim[CB], dl[CB], wmin = kNoLimit;
  int64_t orow[CB];
  bool rvalid[CB];
#pragma unroll
  for (int c = 0; c < CB; ++c) {
    const int row = row0 + 16 * c + lr;
    rvalid[c] = row < nrows;
    const int qi = rvalid[c] ? row / group : 0;
    const int qh = kvh * group + (rvalid[c] ? row % group : 0);
    lim[c] = rvalid[c] ? qi + R.ls - R.lq : -1;
    dl[c] = rvalid[c] && p.doc_lim ? p.doc_lim[R.q0 + qi] : kNoLimit;
    orow[c] = (int64_t)(R.q0 + qi) * p.n_q_heads + qh;
    wmin = min(wmin, dl[c]);
  }
  if (p.doc_lim) {
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) wmin = min(wmin, __shfl_xor(wmin, o));
    wmin = uni(wmin);
  } else {
    wmin = kNoLimit;
  }

  const uint32_t koff =
      (uint32_t)((S::F32 ? lr : 8 * (lr >> 2) + (lr & 3)) * D * (int)sizeof(T) + 16 * lg);
  const uint32_t voff = (uint32_t)(lr * kT * (int)sizeof(T) + 16 * lg);

  const OwnRows own = kSmall ? own_rows<T, D>(p, R, kvh) : OwnRows{};
  Tile<T, D> ta, tb;
  TileInfo ia{}, ib{};
  auto load = [&](int t, bool live, TileInfo &i, Tile<T, D> &x) {
    i = tile_info<T, D>(cur, t);
    if (kSmall && i.own)
      load_own<T, D>(own, i.j0, lr, lg, x);
    else
      load_tile<T, D>(i, kSmall || live ? koff : 0, kSmall || live ? voff : 0, x);
  };
  if (t_begin < t_end) load(t_begin, true, ia, ta);
  uint4 qf[CB][S::KU];
#pragma unroll
  for (int c = 0; c < CB; ++c) {
    const char *q = (const char *)p.q + orow[c] * (D * (int)sizeof(T)) + 16 * lg;
#pragma unroll
    for (int jj = 0; jj < S::KU; ++jj) {
      uint4 v = make_uint4(0, 0, 0, 0);
      if (rvalid[c]) v = *(const uint4 *)(q + 64 * jj);
      qf[c][jj] = v;
    }
  }
  State<T, D, CB> st;
#pragma unroll
  for (int c = 0; c < CB; ++c) {
    st.m[c] = -INFINITY;
    st.l[c] = 0.f;
#pragma unroll
    for (int b = 0; b < S::NB; ++b) st.o[c][b] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  const float sc = p.scale_log2;

  // The loads past the last tile read one line each of it: a branch around
  // them makes the compiler wait for every load in flight where the paths
  // meet (the small form branches anyway, on own tiles).
  for (int t = t_begin; t < t_end; t += 2) {
    if (!kSmall || t + 1 < t_end) load(min(t + 1, t_end - 1), t + 1 < t_end, ib, tb);
    compute_tile<T, D, CB>(ta, ia, qf, st, lg, lim, dl, wmin, sc);
    if (t + 1 >= t_end) break;
    if (!kSmall || t + 2 < t_end) load(min(t + 2, t_end - 1), t + 2 < t_end, ia, ta);
    compute_tile<T, D, CB>(tb, ib, qf, st, lg, lim, dl, wmin, sc);
  }

  const int64_t part0 = part_row - (int64_t)R.q0 * p.n_q_heads;   // partial row of output row 0
  float ltot[CB];
#pragma unroll
  for (int c = 0; c < CB; ++c) ltot[c] = col_sum(st.l[c]);
  // (NaN stays in the maxima; a row whose probabilities sum to NaN sees a NaN
  // score, and no order of its sums changes what it gives)
  float most = 0.f;
#pragma unroll
  for (int c = 0; c < CB; ++c) {
    float mc = 0.f;
#pragma unroll
    for (int b = 0; b < S::NB; ++b)
#pragma unroll
      for (int i = 0; i < 4; ++i) mc = __builtin_elementwise_maximum(mc, fabsf(st.o[c][b][i]));
    most = __builtin_elementwise_maximum(most, ltot[c] == ltot[c] ? mc : 0.f);
  }
  const bool redo = __any(!(most <= kSafeSum));
  if (__builtin_expect(redo, 0)) {
    // the piece anew: kept over the loop above, it would cost it registers
    int block = blockIdx.x;
    asm volatile("" : "+s"(block));
    Piece again;
    if (piece_of<kSmall, kR>(p, links, reqs, order, block, wave, lane, again))
      rows_alone<T, D, kSmall>(p, again, kR, lane, so[wave], kOS, sm[wave], sl[wave]);
    __builtin_amdgcn_wave_barrier();     // its lanes read each other's sums below
  }
  if (__builtin_expect(kpar == 1 && !redo, 1)) {
    // each lane holds 4 consecutive value dims of its rows
#pragma unroll
    for (int c = 0; c < CB; ++c) {
      if (!rvalid[c]) continue;
      if (part_row < 0) {
        const float inv = ltot[c] > 0.f ? 1.f / ltot[c] : 0.f;
        T *out = (T *)p.out + orow[c] * D + 4 * lg;
#pragma unroll
        for (int b = 0; b < S::NB; ++b)
          store4<T>(out + 16 * b, st.o[c][b][0] * inv, st.o[c][b][1] * inv, st.o[c][b][2] * inv,
                    st.o[c][b][3] * inv);
        if (p.lse && lg == 0)
          p.lse[orow[c]] = ltot[c] > 0.f ? log_sum(st.m[c], ltot[c]) : -INFINITY;
      } else {
        const int64_t prow = part0 + orow[c];
        float *po = p.part_o + prow * D + 4 * lg;
#pragma unroll
        for (int b = 0; b < S::NB; ++b)
          store4<float>(po + 16 * b, st.o[c][b][0], st.o[c][b][1], st.o[c][b][2], st.o[c][b][3]);
        if (lg == 0) {
          p.part_m[prow] = partial_max(st.m[c], ltot[c]);
          p.part_l[prow] = ltot[c];
        }
      }
    }
    return;
  }
  // (m, l, O) of rows in LDS to out or the partials: units of 4 value dims idx,
  // idx + step ... of n rows from row `begin` on, the sum of kParts waves' from
  // wave0 on (a constant: their reads of LDS go out together).
  auto write_rows = [&](int idx, int step, int n, int begin, int wave0, auto parts) {
    constexpr int kParts = decltype(parts)::value;
    constexpr int kQ = D / 4;                      // 4-wide units per row
    for (; idx < n * kQ; idx += step) {
      const int rr = idx / kQ, e = idx % kQ * 4;
      const int row = begin + rr;
      if (row >= nrows) break;                     // later units are later rows
      const int w0 = wave0 + rr / kR * kParts, rl = rr % kR;
      float M = -INFINITY, L = 0.f;
#pragma unroll
      for (int w = 0; w < kParts; ++w) M = fmaxf(M, sm[w0 + w][rl]);
      float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int w = 0; w < kParts; ++w) {
        const float mw = sm[w0 + w][rl];
        const float wt = mw == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mw - M);
        const float4 v = *(const float4 *)&so[w0 + w][rl * kOS + e];
        L += wt * sl[w0 + w][rl];
        a.x += wt * v.x;
        a.y += wt * v.y;
        a.z += wt * v.z;
        a.w += wt * v.w;
      }
      const int64_t orw = (int64_t)(R.q0 + row / group) * p.n_q_heads + kvh * group + row % group;
      if (part_row < 0) {
        const float inv = L > 0.f ? 1.f / L : 0.f;
        store4<T>((T *)p.out + orw * D + e, a.x * inv, a.y * inv, a.z * inv, a.w * inv);
        if (p.lse && e == 0)
          p.lse[orw] = L > 0.f ? log_sum(M, L) : -INFINITY;
      } else {
        const int64_t prow = part0 + orw;
        store4<float>(p.part_o + prow * D + e, a.x, a.y, a.z, a.w);
        if (e == 0) {
          p.part_m[prow] = M;
          p.part_l[prow] = L;
        }
      }
    }
  };
  if (kpar == 1) {
    write_rows(lane, 64, kR, row0, wave, std::integral_constant<int, 1>());
    return;
  }
  // merge the kpar parts of every row block through LDS
  if (!redo) {
#pragma unroll
    for (int c = 0; c < CB; ++c) {
      float *o = &so[wave][(16 * c + lr) * kOS + 4 * lg];
#pragma unroll
      for (int b = 0; b < S::NB; ++b)
        store4<float>(o + 16 * b, st.o[c][b][0], st.o[c][b][1], st.o[c][b][2], st.o[c][b][3]);
      if (lg == 0) {
        sm[wave][16 * c + lr] = partial_max(st.m[c], ltot[c]);
        sl[wave][16 * c + lr] = ltot[c];
      }
    }
  }
  __syncthreads();
  if (kpar == 2)
    write_rows(threadIdx.x, 64 * kWaves, 2 * kR, wg_row0, 0, std::integral_constant<int, 2>());
  else
    write_rows(threadIdx.x, 64 * kWaves, kR, wg_row0, 0, std::integral_constant<int, 4>());
}

// Two waves per SIMD, one for the widest fp32 heads (two tiles in flight of
// 64 registers each for K and V).
template <typename T, int D>
constexpr int kMinWaves = D * sizeof(T) > 256 ? 1 : 2;

template <typename T, int D, int CB>
__global__ __launch_bounds__(64 * kWaves, (kMinWaves<T, D>)) void link_stream_kernel(LinkParams p) {
  stream_body<T, D, CB, false>(p, (const_links)p.links, nullptr, nullptr);
}

// The tables are read where they are, in the kernel arguments.
struct SmallArgs {
  LinkParams p;
  SmallTabs t;
};
template <typename T, int D, int CB>
__global__ __launch_bounds__(64 * kWaves, (kMinWaves<T, D>)) void link_small_kernel(SmallArgs a) {
  typedef __attribute__((address_space(4))) const char *const_bytes;
  const const_bytes arg = (const_bytes)__builtin_amdgcn_kernarg_segment_ptr();
  stream_body<T, D, CB, true>(a.p, (const_links)(arg + offsetof(SmallArgs, t.links)),
                              (const_reqs)(arg + offsetof(SmallArgs, t.reqs)),
                              (const_ints)(arg + offsetof(SmallArgs, t.order)));
}

// f(T{}, constant D, constant CB) for the shape's instantiation.
template <typename F>
hipError_t pick(int dtype, int d, int cb, F f) {
  auto by_cb = [&](auto t, auto dc) {
    if (cb == 1) return f(t, dc, std::integral_constant<int, 1>());
    if (cb == 2) return f(t, dc, std::integral_constant<int, 2>());
    if constexpr (sizeof(t) == 2) return f(t, dc, std::integral_constant<int, 4>());
    return hipErrorInvalidValue;
  };
  if (dtype == 0) {
    if (d == 32) return by_cb(float(), std::integral_constant<int, 32>());
    if (d == 64) return by_cb(float(), std::integral_constant<int, 64>());
    return by_cb(float(), std::integral_constant<int, 128>());
  }
  if (d == 32) return by_cb(uint16_t(), std::integral_constant<int, 32>());
  return by_cb(uint16_t(), std::integral_constant<int, 64>());
}
// Whether a small call is built for the shape: not where the in-place own
// tiles would take the registers past their budget (wide heads and many
// column blocks; such calls have little to gain).
constexpr bool small_built(int esz, int d, int cb) { return cb * d * esz <= 512 && cb <= 2; }

unsigned stream_blocks(const LinkParams &p, int64_t units) {
  return (unsigned)unit_blocks(units, p.nrb, p.n_xcd, p.spread);
}

}  // namespace

bool stream_supported(int dtype, int d_k, int d_v) {
  if (d_k != d_v) return false;
  return d_k == 32 || d_k == 64 || (d_k == 128 && dtype == 0);
}

StreamShape stream_shape(int dtype, int d, int max_rows, bool small) {
  int cb = max_rows <= 16 ? 1 : max_rows <= 32 || dtype == 0 ? 2 : 4;
  if (small)
    while (!small_built(dtype == 0 ? 4 : 2, d, cb)) cb /= 2;
  StreamShape s;
  // one workgroup (a wave per SIMD) for the widest fp32 heads, see kMinWaves;
  // the others hold at least two
  s.per_cu = d * (dtype == 0 ? 4 : 2) > 256 ? 1 : 2;
  s.rows = 16 * cb;
  const int blocks = (max_rows + s.rows - 1) / s.rows;
  s.kpar = blocks <= 1 ? 4 : blocks == 2 ? 2 : 1;
  return s;
}

// Measured against the vector-ALU kernel these calls ran before (kernel time,
// one MI355X): fp32 8/2 heads x 64, 12 ragged requests of 20..130 tokens over
// 3..10 links 395 -> 53 us; bf16 32/8 x 64, 8 requests of 30..300 tokens
// 3320 -> 139 us. At 512 tokens x 16 links x 1024, batch 4 (no ragged edges):
// bf16 d 64 584 TFLOP/s (876 with the second product of the lo parts), fp32
// 109 TFLOP/s of the 154 a large library product reaches. Decode, 64 requests
// x 16 links x 1024: bf16 5.9 TB/s, fp32 5.6 TB/s.
hipError_t launch_link_stream(const LinkParams &p, int dtype, int rows, hipStream_t st,
                              const char **name) {
  *name = dtype == 0 ? "link_stream_kernel<float>" : "link_stream_kernel<bf16>";
  return pick(dtype, p.d_k, rows / 16, [&](auto t, auto dc, auto cb) {
    hipLaunchKernelGGL((link_stream_kernel<decltype(t), decltype(dc)::value, decltype(cb)::value>),
                       dim3(stream_blocks(p, (int64_t)p.n_items * p.n_kv_heads)),
                       dim3(64 * kWaves), 0, st, p);
    return hipGetLastError();
  });
}

hipError_t launch_link_stream_small(const LinkParams &p, const SmallTabs &tabs, int dtype, int rows,
                                    hipStream_t st, const char **name) {
  *name = dtype == 0 ? "link_small_kernel<float,stream>" : "link_small_kernel<bf16,stream>";
  return pick(dtype, p.d_k, rows / 16, [&](auto t, auto dc, auto cb) {
    constexpr int kD = decltype(dc)::value, kCB = decltype(cb)::value;
    if constexpr (small_built(sizeof(t), kD, kCB)) {
      hipLaunchKernelGGL((link_small_kernel<decltype(t), kD, kCB>),
                         dim3(stream_blocks(p, (int64_t)p.batch * p.n_kv_heads * p.num_splits)),
                         dim3(64 * kWaves), 0, st, SmallArgs{p, tabs});
      return hipGetLastError();
    }
    return hipErrorInvalidValue;
  });
}

}  // namespace pic
