// Internal declarations shared by the host planner and the HIP kernels.
// Not part of the C ABI (include/pic.h is).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace pic {

// Keys per attention tile. Every chunk slot in the pool is padded to a
// multiple of it (zero rows), so a tile never straddles two chunks and the
// pool's rows stay 16-byte aligned.
constexpr int kTile = 64;

// Layout of one chunk slot with padded length lp (elements of the store's
// dtype):
//   GQA  K block  [n_kv_heads][lp][d_k]    (head-major, token rows)
//        V block  [n_kv_heads][lp / 32][d_v][32]
//                                          (transposed in panels of 32 tokens:
//                                          value dim = row of a panel, its 32
//                                          tokens contiguous)
//   MLA  K block  [lp][d_k]                (value = first d_v of each row)
// The transposed V lets a matrix-core operand read 8 consecutive keys of one
// value column with a single 16-byte load; the panels keep the rows of a
// 32-key tile together, so a 32-key tile reads whole 128-byte lines (two
// bf16 rows, or one fp32 row) and a 64-key tile is one contiguous block. A
// request's own KV is laid out the same way (in the call's workspace) before
// the attention kernel runs, so every key tile of a request -- document or
// own -- is read alike.
constexpr int kPanel = 32;

// Element offset of value dim e of token t (relative to the slot's first
// token) of head h in a V block with padded length lp.
__host__ __device__ __forceinline__ int64_t vt_offset(int64_t h, int64_t e, int64_t t, int64_t lp,
                                                     int64_t d_v) {
  return h * d_v * lp + (t / kPanel) * (d_v * kPanel) + e * kPanel + (t % kPanel);
}

// A per-row limit on the visible linked rows that no request reaches.
constexpr int kNoLimit = 1 << 30;

struct LinkEntry {        // one link of one request, in link order
  const void *k;          // K block of the slot
  const void *v;          // GQA: V block; MLA: same as k
  int32_t len;            // tokens; the link spans ceil(len / kTile) tiles
  int32_t lp;             // row stride of its K / V^T blocks in tokens (multiple of kTile)
  int32_t tile0;          // index of the link's first tile within the request
  int32_t tok0;           // index of the link's first token within the request
};

struct ReqEntry {
  int32_t link0, nlinks;  // links[link0 .. link0+nlinks); the own KV, if any, is the last
  int32_t q0, lq;         // query rows q0 .. q0+lq of q / out
  int32_t s0, ls;         // own rows s0 .. s0+ls of k_self / v_self (ls = 0: none)
  int32_t doc_tiles;      // tiles over the linked documents (own tiles follow)
  int32_t tiles;          // doc_tiles + ceil(ls / kTile)
};

// Tiles of a request that hold a key visible to query token q_last or any
// earlier one: every document tile, then the own tiles up to the one holding
// own key q_last + ls - lq (the causal limit, bottom-right aligned).
__host__ __device__ __forceinline__ int visible_tiles(const ReqEntry &r, int q_last) {
  const int own_last = q_last + r.ls - r.lq;
  return own_last >= 0 ? (r.doc_tiles + own_last / kTile + 1 < r.tiles
                              ? r.doc_tiles + own_last / kTile + 1
                              : r.tiles)
                       : r.doc_tiles;
}

// One piece of a request's keys: a kernel's unit of work for one kv head (and
// row block). Holds all that a workgroup needs before its first key load, so
// that load waits for one table read (the request order, the request and a
// walk over its links were three and more dependent ones). The link fields
// are those of the entry that holds tile t_begin; later links follow at
// links[link + 1] ... (for the decode kernel, which masks no linked rows, tok0
// is the request's first own row)
struct WorkItem {
  const void *k, *v;
  int32_t len, lp, tile0, tok0;
  int32_t link;
  int32_t t_begin, t_end; // tiles of the piece, in the kernel's tile size
  int32_t q0, lq, ls, doc_tiles;
  int32_t part;           // first partial row of the piece (row i of the request
                          // at part + i); -1: the request is not split
};
static_assert(sizeof(WorkItem) == 64, "one 64-byte line per item");

// A request's split partials for the combine: rows row0 .. row0 + rows of
// out, piece s of row i at partial row part0 + s * rows + i.
struct CombineEntry {
  int32_t row0, rows, part0, splits;
};

struct LinkParams {
  const LinkEntry *links;
  const WorkItem *items;  // NULL for the vector-ALU and small-call kernels
  const ReqEntry *reqs;
  const int32_t *order;   // requests, heaviest first
  const CombineEntry *comb;   // per request (NULL: num_splits pieces of every row)
  const void *q;
  const void *k_self;
  const void *v_self;
  void *out;
  float *lse;
  float *part_o;          // split partials: [partial row][d_v] unnormalised
  float *part_m;          // [partial row] running max (log2 domain)
  float *part_l;          // [partial row] running sum
  const int32_t *doc_lim; // per query token: linked rows it sees (NULL: all of them)
  int32_t batch;
  int32_t n_items;
  int32_t n_q_heads;
  int32_t n_kv_heads;
  int32_t group;          // n_q_heads / n_kv_heads
  int32_t d_k;
  int32_t d_v;
  int32_t total_q;        // Tq
  int32_t num_splits;     // most pieces of a request (1: nothing to combine)
  int32_t nrb;            // row blocks per (request, kv head)
  int32_t max_rows;       // most rows of one (request, kv head)
  int32_t n_groups;       // batch * n_kv_heads
  int32_t spread;         // matrix-core kernels: row blocks of one unit on all XCDs (1, 2)
  int32_t n_xcd;          // accelerator dies (XCDs) of the device, each with its own L2
  int32_t skip_empty;     // values of partials with m = -inf are not written
  int32_t even;           // all requests have as many tiles, rows and pieces
  int32_t gang;           // MLA kernel: consecutive row blocks on one XCD (planned: its CUs)
  int32_t kpar;           // stream kernel: key parts within a workgroup (1, 2 or 4)
  float scale_log2;       // softmax_scale * log2(e)
};

// Shape of the current device: compute units and XCDs. Workgroups with
// consecutive ids are dispatched round-robin to the XCDs, so a kernel that
// wants some of them to share an L2 maps ids with the XCD count.
struct DevShape {
  int32_t cus;
  int32_t xcds;
};
DevShape device_shape();

// Work mapping of the matrix-core kernels: workgroup b of the grid takes row
// block rb of unit u (item x kv head). Consecutive workgroups go round-robin
// to the XCDs; the row blocks of one unit read the same keys, so they share
// an XCD and its L2 and are dispatched back to back. Where that would leave
// XCDs idle (few units, or a last round of them that fills few XCDs: more
// than a quarter of the places empty), the row blocks of every unit spread
// over all XCDs instead: block 0 of every unit first, or (spread 2: calls with
// per-query limits) the last one, whose rows see the most. (The stream kernel
// spreads them always, see apply_splits.)
inline bool spread_units(int64_t units, int32_t nrb, int32_t n_xcd) {
  return nrb > 1 && 4 * ((units + n_xcd - 1) / n_xcd * n_xcd) > 5 * units;
}
inline int64_t unit_blocks(int64_t units, int32_t nrb, int32_t n_xcd, bool spread) {
  return spread ? units * nrb : (units + n_xcd - 1) / n_xcd * n_xcd * nrb;
}
struct UnitBlock {
  int32_t u, rb;
};
__device__ __forceinline__ UnitBlock unit_of_block(int32_t b, int32_t nrb, int32_t n_xcd,
                                                   int32_t spread, int32_t units) {
  if (spread) return UnitBlock{b % units, spread == 2 ? nrb - 1 - b / units : b / units};
  const int32_t xcd = b % n_xcd, j = b / n_xcd;
  return UnitBlock{xcd + n_xcd * (j / nrb), j % nrb};
}

// Items and tables are read through the constant address space: every lookup
// is a scalar load.
typedef __attribute__((address_space(4))) const LinkEntry *const_links;
typedef __attribute__((address_space(4))) const WorkItem *const_items;
__device__ __forceinline__ WorkItem load_item(const WorkItem *items, int32_t i) {
  const_items p = (const_items)items + i;
  WorkItem w;
  w.k = p->k;
  w.v = p->v;
  w.len = p->len;
  w.lp = p->lp;
  w.tile0 = p->tile0;
  w.tok0 = p->tok0;
  w.link = p->link;
  w.t_begin = p->t_begin;
  w.t_end = p->t_end;
  w.q0 = p->q0;
  w.lq = p->lq;
  w.ls = p->ls;
  w.doc_tiles = p->doc_tiles;
  w.part = p->part;
  return w;
}
__device__ __forceinline__ ReqEntry item_request(const WorkItem &w) {
  ReqEntry R{};
  R.q0 = w.q0;
  R.lq = w.lq;
  R.ls = w.ls;
  R.doc_tiles = w.doc_tiles;
  R.tiles = w.doc_tiles + (w.ls + kTile - 1) / kTile;
  return R;
}

// The running max a partial (m, l, O) is stored with: -inf only where it holds
// no key, which is what the combine passes over. A NaN sum stays in the merge
// (the max beside it is -inf where every score is NaN).
__device__ __forceinline__ float partial_max(float m, float l) {
  return l == 0.f ? -INFINITY : m == -INFINITY ? 0.f : m;
}

// ln(2^m l), the log-sum-exp of a running max and its sum, rounded once. (m +
// log2 l) ln 2 in fp32 rounds three times, and where the max lags behind, as in
// the streaming kernel, l is larger and its logarithm coarser: fp32 lse was up
// to a tenth further from 64 bits than the vector kernel's.
__device__ __forceinline__ float log_sum(float m, float l) {
  int e;
  const float f = frexpf(l, &e);
  return (float)(((double)m + e) * 0.69314718055994530942 + (double)logf(f));
}

// All-lane max / sum of a wave without LDS round trips: DPP moves inside
// each 16-lane row (lane ^ 1, lane ^ 2 by quad permutes, then the mirrors
// of each 8-lane half and of the row), then lanes l ^ 16 and l ^ 32 by the
// permlane swaps. Every lane ends with the wave's result.
template <int kCtrl>
__device__ __forceinline__ float dpp_mov(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), kCtrl, 0xF, 0xF, false));
}
__device__ __forceinline__ float wave_max(float x) {
  x = fmaxf(x, dpp_mov<0xB1>(x));    // quad_perm [1,0,3,2]
  x = fmaxf(x, dpp_mov<0x4E>(x));    // quad_perm [2,3,0,1]
  x = fmaxf(x, dpp_mov<0x141>(x));   // row_half_mirror
  x = fmaxf(x, dpp_mov<0x140>(x));   // row_mirror
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float wave_sum(float x) {
  x += dpp_mov<0xB1>(x);
  x += dpp_mov<0x4E>(x);
  x += dpp_mov<0x141>(x);
  x += dpp_mov<0x140>(x);
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Epilogue stores of the matrix-core kernels. After the 32x32 value products
// lane (n = l % 32, g = l / 32) holds row n, value dims 32 d + 8 j + 4 g ..+3
// of a 32-row x 128-dim block, so a store straight from the registers covers
// 32 rows x 16 bytes (bf16) or x 32 bytes (fp32) of lines 128 bytes long. The
// block goes through LDS instead (8 KB per wave, 16-byte chunks XOR-swizzled
// by the row, free of bank conflicts) and leaves as whole 256-byte row pieces,
// 4 rows per instruction. row: the output row of this lane's row n (any
// value for rows past nvalid); out: its row 0, first of the block's dims.
typedef float acc32x32 __attribute__((ext_vector_type(16)));
constexpr uint32_t kStoreBytes = 8192;      // LDS per wave
typedef uint32_t u32x4v __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2v __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) u32x4v *lds_units;
typedef __attribute__((address_space(3))) u32x2v *lds_halves;
typedef float f32x4v __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x4v __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void store_block_units(lds_units lds, int lane, int nvalid, int row,
                                                  char *out, int64_t row_bytes) {
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int r = 4 * k + (lane >> 4), c = lane & 15;
    const u32x4v u = lds[r * 16 + (c ^ (r & 15))];
    const int at = __shfl(row, r);
    if (r < nvalid) *(u32x4v *)(out + at * row_bytes + 16 * c) = u;
  }
}
__device__ __forceinline__ void store_block_bf16(const acc32x32 &o0, const acc32x32 &o1,
                                                 const acc32x32 &o2, const acc32x32 &o3, float inv,
                                                 lds_units lds, int lane, int nvalid, int row,
                                                 uint16_t *out, int64_t stride) {
  const int n = lane & 31, g = lane >> 5;
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    const acc32x32 &o = d == 0 ? o0 : d == 1 ? o1 : d == 2 ? o2 : o3;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      bf16x4v v4;
#pragma unroll
      for (int x = 0; x < 4; ++x) v4[x] = (__bf16)(o[j * 4 + x] * inv);
      ((lds_halves)lds)[(n * 16 + ((4 * d + j) ^ (n & 15))) * 2 + g] = __builtin_bit_cast(u32x2v, v4);
    }
  }
  store_block_units(lds, lane, nvalid, row, (char *)out, stride * 2);
}
__device__ __forceinline__ void store_block_f32(const acc32x32 &o0, const acc32x32 &o1,
                                                const acc32x32 &o2, const acc32x32 &o3, lds_units lds,
                                                int lane, int nvalid, int row, float *out,
                                                int64_t stride) {
  const int n = lane & 31, g = lane >> 5;
#pragma unroll
  for (int h = 0; h < 2; ++h) {       // dims 64 h .. 64 h + 63
#pragma unroll
    for (int d = 0; d < 2; ++d) {
      const acc32x32 &o = h == 0 ? (d == 0 ? o0 : o1) : (d == 0 ? o2 : o3);
#pragma unroll
      for (int j = 0; j < 4; ++j)
        lds[n * 16 + ((8 * d + 2 * j + g) ^ (n & 15))] = __builtin_bit_cast(
            u32x4v, (f32x4v){o[j * 4], o[j * 4 + 1], o[j * 4 + 2], o[j * 4 + 3]});
    }
    store_block_units(lds, lane, nvalid, row, (char *)(out + 64 * h), stride * 4);
  }
}

// Launchers (each returns the launch status).

// One run of a put chunk: token-major sources [layer][n_tokens..][heads][d]
// into the run's K block and V block of every layer (src_v NULL for MLA).
struct PutParams {
  const char *src_k, *src_v;      // the run's first token, layer 0
  char *dst_k, *dst_v;            // the run's blocks in layer 0
  int64_t src_k_layer, src_v_layer, layer_bytes;   // bytes from layer to layer
  int32_t n_tokens, lp, heads, d_k, d_v, esz;
  int32_t rows_blocks;            // set by launch_put
};
hipError_t launch_put(PutParams pp, int32_t n_layers, hipStream_t st);
hipError_t launch_gather(const LinkEntry *links, int32_t n_links, int64_t total_tokens,
                         int32_t heads, int32_t d_k, int32_t d_v, int32_t mla, int32_t esz,
                         void *k_out, void *v_out, hipStream_t st);

// Page copies of a derived chunk (kernel argument): pages of 64 tokens, kv
// head 0 of layer 0 (head h at + h * lp * width elements); v NULL for MLA.
struct PageCopy {
  const char *src_k, *src_v;
  char *dst_k, *dst_v;
  int32_t src_lp, dst_lp;
};
constexpr int kCopyPages = 64;
struct PageCopies {
  PageCopy page[kCopyPages];
  int64_t layer_bytes;
  int32_t heads, d_k, d_v, esz;
};
hipError_t launch_copy_pages(const PageCopies &c, int32_t n, int32_t n_layers, hipStream_t st);

// A view of a chunk in one layer, for rows written into it: its K rows and V
// panels of head 0 (head h at + h * lp * width elements; v NULL for MLA)
// from chunk token tok0 on.
struct RowView {
  void *k, *v;
  int32_t lp, tok0;
};
// Kernel argument of a row write: up to kRows rows in up to kWriteViews
// views (ascending tokens).
constexpr int kWriteViews = 16, kWriteRowsFew = 128, kWriteRowsMost = 768;
template <int kRows>
struct WriteRows {
  RowView view[kWriteViews];
  int32_t n_views;
  int32_t row[kRows];
};
// Scatters token-major rows src_k [n][heads][d_k] (and src_v [n][heads][d_v]
// unless the views' v are NULL) to chunk tokens rows[0 .. n), n <=
// kWriteRowsMost, n_views <= kWriteViews.
hipError_t launch_write_rows(const RowView *views, int32_t n_views, const int32_t *rows, int32_t n,
                             const void *src_k, const void *src_v, int32_t heads, int32_t d_k,
                             int32_t d_v, int32_t esz, hipStream_t st);

// Copies bytes (a multiple of 16) from a host-mapped buffer to the device.
hipError_t launch_table_copy(const void *src, void *dst, int64_t bytes, hipStream_t st);

// The dense MLA projections around the latent link (see pic.h).
hipError_t launch_mla_absorb_q(const void *q, const void *w_uk_t, void *q_out, int32_t n_tokens,
                               int32_t n_heads, const DevShape &ds, hipStream_t st);
hipError_t launch_mla_up_v(const void *o_lat, const void *w_uv, void *out, int32_t n_tokens,
                           int32_t n_heads, const DevShape &ds, hipStream_t st);
// The call's prologue: lays out the own KV of every request (token-major
// k_self / v_self) like a chunk slot at its own link (the request's last
// link), zero-padded to lp, in `work` (when max_own_lp > 0) and copies copy_bytes of tables from
// copy_src to copy_dst (when copy_bytes > 0). The layout takes each
// request's own rows and slot from `own` (host, batch entries, batch <=
// kOwnArgs: passed as kernel arguments, so it does not wait for a read of
// the tables over PCIe from the staging buffer), or, when own is NULL,
// from the tables at links / reqs.
struct OwnArg {
  int32_t s0, ls;     // own rows s0 .. s0+ls of k_self / v_self
  int64_t off;        // slot offset in the workspace (K block, then V^T block)
};
constexpr int kOwnArgs = 128;
hipError_t launch_prologue(const LinkParams &p, const LinkEntry *links, const ReqEntry *reqs,
                           int32_t mla, int32_t esz, int32_t max_own_lp, const OwnArg *own,
                           const void *work, const void *copy_src, void *copy_dst,
                           int64_t copy_bytes, hipStream_t st);

// Generic vector-ALU link attention: any d_k <= 576, d_v <= 512, fp32 or bf16.
hipError_t launch_link_valu(const LinkParams &p, int dtype, int mla, hipStream_t st,
                            const char **name);
int valu_rows_per_block();

// bf16 GQA link attention on MFMA, d_k = d_v = 128 (prefill-shaped).
hipError_t launch_link_mfma_d128(const LinkParams &p, hipStream_t st, const char **name);
int mfma_d128_rows_per_block();
int mfma_d128_blocks_per_cu();   // resident workgroups per CU (2 waves per SIMD)

// bf16 GQA decode-shaped link attention, d_k = d_v = 128, at most
// decode_d128_max_rows() rows per (request, kv head); one wave per split.
hipError_t launch_link_decode_d128(const LinkParams &p, hipStream_t st, const char **name);
int decode_d128_max_rows();

// fp32 GQA (d_k = d_v in {32, 64, 128}) and narrow bf16 GQA ({32, 64}) link
// attention on the matrix cores, prefill- and decode-shaped. stream_shape:
// rows per wave and key parts per workgroup of a call whose largest request
// has max_rows rows per kv head; a workgroup covers rows * 4 / kpar rows.
bool stream_supported(int dtype, int d_k, int d_v);
struct StreamShape {
  int32_t rows, kpar;
  int32_t per_cu;         // resident workgroups per CU that a call is planned with
};
StreamShape stream_shape(int dtype, int d, int max_rows, bool small);
hipError_t launch_link_stream(const LinkParams &p, int dtype, int rows, hipStream_t st,
                              const char **name);

// bf16 MLA (absorbed) link attention: one 576-wide latent kv head, values
// are the first 512 entries of each latent row.
hipError_t launch_link_mla(LinkParams p, hipStream_t st, const char **name);
int mla_rows_per_block();

// Achievable-peak microbenchmarks (out: peak_out_floats() floats of scratch).
int64_t peak_out_floats();
double peak_mfma_flops(int32_t iters);
hipError_t launch_peak_mfma(float *out, int32_t iters, hipStream_t st);
hipError_t launch_peak_read(const void *src, int64_t bytes, float *out, hipStream_t st);
hipError_t launch_peak_write(void *dst, int64_t bytes, hipStream_t st);

// The library's static device scratch (a file-scope array, no allocation):
// its size, and its address on the current device (resolved once per
// device). Used by the entry points that must not allocate.
// kStaticScratchSlack: room beyond what a call is charged for, for its work
// items (64 B each).
constexpr size_t kStaticScratchBytes = size_t(64) << 20;
constexpr size_t kStaticScratchSlack = size_t(8) << 20;
constexpr int kMaxDevices = 64;
hipError_t static_scratch(void **out);

// Log-sum-exp merge of split partials into out / lse.
// max_rows: most rows of one p.comb entry (unused when p.comb is NULL).
hipError_t launch_combine(const LinkParams &p, int dtype, int32_t max_rows, hipStream_t st);

// Tables of a small call (vector-ALU or streaming kernel), passed by value as a kernel
// argument: the call then needs neither the table copy nor the own-KV
// layout of the prologue (see link_small_kernel).
constexpr int kSmallLinks = 32, kSmallReqs = 8;
struct SmallTabs {
  LinkEntry links[kSmallLinks];
  ReqEntry reqs[kSmallReqs];
  int32_t order[kSmallReqs];
};
hipError_t launch_link_small(const LinkParams &p, const SmallTabs &t, int dtype, int mla,
                             hipStream_t st, const char **name);
hipError_t launch_link_stream_small(const LinkParams &p, const SmallTabs &t, int dtype, int rows,
                                    hipStream_t st, const char **name);

// Tables of a lean small call (link_lean_kernel): requests in dispatch
// order, and for every tile of every request the link that holds it
// (relative to the request's first link), so a workgroup finds its tiles
// with one table read instead of a walk over the links.
constexpr int kLeanTiles = 256;
struct LeanTabs {
  LinkEntry links[kSmallLinks];
  ReqEntry reqs[kSmallReqs];          // reqs[i]: the i-th request in dispatch order
  int32_t tile_base[kSmallReqs];      // first tile_link entry of reqs[i]
  uint8_t tile_link[kLeanTiles];
};
// GQA shapes the lean kernel is built for: d_k = d_v = d in {32, 64, 128}
// for fp32, {32, 64} for bf16, and a power-of-two query group.
bool lean_supported(int dtype, int d_k, int d_v, int group);
hipError_t launch_link_lean(const LinkParams &p, const LeanTabs &t, int dtype, hipStream_t st,
                            const char **name);

}  // namespace pic
