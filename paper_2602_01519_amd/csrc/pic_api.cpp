// C ABI of the link-stage attention library: the chunk store (pool +
// hash table + bump allocator), the per-call link planner and its staging of
// the chunk table, kernel selection, and kernel timing.
#include "../../include/pic.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <functional>
#include <map>
#include <initializer_list>
#include <mutex>
#include <string>
#include <unordered_map>
#include <vector>

#include "pic_internal.hpp"

namespace pic {
size_t valu_lds_bytes_for(int esz, int mla, int d_k, int d_v);
}

using namespace pic;

namespace {

thread_local std::string g_err;

pic_status fail(pic_status st, const char *fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_err = buf;
  return st;
}

pic_status hip_fail(hipError_t e, const char *what) {
  return fail(PIC_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
}

#define HIP_TRY(expr, what)                 \
  do {                                      \
    hipError_t e_ = (expr);                 \
    if (e_ != hipSuccess) return hip_fail(e_, what); \
  } while (0)

// Restores the caller's current device on scope exit.
struct DeviceGuard {
  int prev = -1;
  bool ok = true, switched = false;
  explicit DeviceGuard(int dev) {
    if (hipGetDevice(&prev) != hipSuccess) { ok = false; return; }
    if (prev != dev) {
      switched = true;
      if (hipSetDevice(dev) != hipSuccess) ok = false;
    }
  }
  ~DeviceGuard() {
    if (switched && prev >= 0) (void)hipSetDevice(prev);
  }
};

// The pool is a sequence of 64-token pages (one attention tile each). A
// chunk occupies runs of consecutive pages -- one run whenever a free run
// is long enough -- and each run holds a piece of the chunk laid out like a
// chunk of its own (K [H][run tokens][d_k], then V^T [H][d_v][run tokens]),
// so a piece is one link-table entry and the kernels need no page table.
// Such a run of pages is a block; a chunk is a list of views of blocks
// (pages skip .. of the block), in token order. A chunk made by
// pic_store_derive views its base's blocks for the pages it shares with
// it, so blocks are reference-counted by the chunks that view them.
struct Run {
  int64_t page0;        // the block's first page
  int32_t pages;        // the block's pages (its row stride is pages * 64 tokens)
  int32_t tok0;         // first chunk token held by the view
  int32_t ntok;         // chunk tokens held by the view
  int32_t skip = 0;     // pages of the block before the view's first page
};

struct Slot {
  int64_t len;
  std::vector<Run> runs;
  int64_t plan_refs = 0;   // live link plans that link this chunk
  bool derived = false;    // made by pic_store_derive (rows may be written)
};

// Pinned host table + device copy + completion event. The planner writes a
// call's chunk/request tables into one slot, copies them to the device on
// the call's stream, and records the event after the call's last kernel; a
// slot is reused only after its event has completed.
// A call's workspace (own-KV slots, split partials) belongs to its slot
// too, so calls in flight on different streams never share one.
struct Stage {
  void *host = nullptr;
  void *host_dev = nullptr;     // device-visible address of host
  void *dev = nullptr;
  size_t cap = 0;
  void *work = nullptr;
  size_t work_cap = 0;
  hipEvent_t done = nullptr;
  bool pending = false;
};

constexpr int kRing = 8;

struct ProfState {
  std::mutex mu;
  bool on = false;
  int32_t every = 1;       // time one launch in `every`
  int64_t seen = 0;        // launches since the last begin
  std::vector<std::pair<hipEvent_t, hipEvent_t>> events;
  std::vector<std::pair<hipEvent_t, hipEvent_t>> spare;
  std::string name;
};
ProfState g_prof;

inline int64_t round_up(int64_t x, int64_t m) { return (x + m - 1) / m * m; }

}  // namespace

namespace pic {
// Queried once per device: compute units, and XCDs (one when the runtime
// does not report them, e.g. a partition that exposes a single die).
DevShape device_shape() {
  static std::mutex mu;
  static std::unordered_map<int, DevShape> cache;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return DevShape{256, 8};
  std::lock_guard<std::mutex> g(mu);
  auto it = cache.find(dev);
  if (it != cache.end()) return it->second;
  int cus = 0, xcds = 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      cus <= 0)
    cus = 256;
  if (hipDeviceGetAttribute(&xcds, hipDeviceAttributeNumberOfXccs, dev) != hipSuccess || xcds <= 0)
    xcds = 1;
  (void)hipGetLastError();
  const DevShape ds{cus, xcds};
  cache.emplace(dev, ds);
  return ds;
}
}  // namespace pic

struct pic_store {
  pic_store_desc desc{};
  int device = 0;
  int esz = 2;
  char *pool = nullptr;
  int64_t capacity = 0;          // padded tokens
  int64_t used = 0;              // tokens of allocated pages
  std::map<int64_t, int64_t> free_runs;   // page0 -> pages, coalesced
  std::unordered_map<int64_t, int32_t> block_refs;   // block page0 -> chunks viewing it
  std::vector<int32_t> page_refs;                     // page -> chunks viewing it
  // runs of removed chunks, reusable once the event (recorded on the
  // remover's stream) has completed
  std::vector<std::pair<hipEvent_t, std::vector<Run>>> pending;
  int32_t n_layers = 1;
  int64_t layer_bytes = 0;       // bytes of one layer's pool; layer l of a slot is l * layer_bytes on
  int64_t live_plans = 0;
  int64_t k_tok_elems = 0;       // K elements per padded token (all heads)
  int64_t v_tok_elems = 0;       // V elements per padded token (GQA)
  std::unordered_map<uint64_t, Slot> map;
  Stage ring[kRing];
  int next = 0;
  DevShape shape{256, 8};        // compute units and XCDs of the store's device
  bool imported = false;         // pool mapped from another process (read-only)
  // request order of the last multi-round d128 prefill call and its key
  // (the request shapes; see balance_order_d128)
  std::vector<int32_t> order_key, order_memo;
};

namespace {

pic_status stage_acquire(pic_store *s, size_t bytes, Stage **out) {
  Stage &st = s->ring[s->next];
  s->next = (s->next + 1) % kRing;
  if (st.pending) {
    HIP_TRY(hipEventSynchronize(st.done), "hipEventSynchronize(stage)");
    st.pending = false;
  }
  // Completion only (the host waits for the copy out of the staging buffer
  // to be done): no system-scope fence, which would write back and
  // invalidate caches after every call.
  if (!st.done)
    HIP_TRY(hipEventCreateWithFlags(&st.done, hipEventDisableTiming | hipEventDisableSystemFence),
            "hipEventCreate");
  if (st.cap < bytes) {
    if (st.host) (void)hipHostFree(st.host);
    if (st.dev) (void)hipFree(st.dev);
    st.host = st.dev = nullptr;
    st.cap = 0;
    size_t cap = std::max<size_t>(round_up((int64_t)bytes, 4096), 64 * 1024);
    HIP_TRY(hipHostMalloc(&st.host, cap, hipHostMallocDefault), "hipHostMalloc(stage)");
    HIP_TRY(hipHostGetDevicePointer(&st.host_dev, st.host, 0), "hipHostGetDevicePointer(stage)");
    HIP_TRY(hipMalloc(&st.dev, cap), "hipMalloc(stage)");
    st.cap = cap;
  }
  *out = &st;
  return PIC_OK;
}

// Grows the workspace of an acquired staging slot (whose previous call has
// completed, so the old buffer is free).
pic_status ensure_work(Stage *st, size_t bytes) {
  if (st->work_cap >= bytes) return PIC_OK;
  if (st->work) {
    (void)hipFree(st->work);
    st->work = nullptr;
    st->work_cap = 0;
  }
  size_t cap = round_up((int64_t)bytes, 1 << 20);
  HIP_TRY(hipMalloc(&st->work, cap), "hipMalloc(workspace)");
  st->work_cap = cap;
  return PIC_OK;
}

// Returns a run of pages to the free map, merging it with free neighbours.
void free_run(pic_store *s, int64_t page0, int64_t pages) {
  auto next = s->free_runs.lower_bound(page0);
  if (next != s->free_runs.end() && next->first == page0 + pages) {
    pages += next->second;
    next = s->free_runs.erase(next);
  }
  if (next != s->free_runs.begin()) {
    auto prev = std::prev(next);
    if (prev->first + prev->second == page0) {
      prev->second += pages;
      return;
    }
  }
  s->free_runs.emplace(page0, pages);
}

// Moves the runs of removed chunks whose readers have finished into the
// free map; with wait, first waits for all of them.
pic_status reclaim(pic_store *s, bool wait) {
  std::vector<std::pair<hipEvent_t, std::vector<Run>>> keep;
  for (auto &pr : s->pending) {
    hipError_t e = wait ? hipEventSynchronize(pr.first) : hipEventQuery(pr.first);
    if (e == hipErrorNotReady) {
      keep.push_back(std::move(pr));
      continue;
    }
    if (e != hipSuccess) return hip_fail(e, "removed-chunk event");
    (void)hipEventDestroy(pr.first);
    for (const Run &r : pr.second) {
      free_run(s, r.page0, r.pages);
      s->used -= (int64_t)r.pages * kTile;
    }
  }
  s->pending.swap(keep);
  return PIC_OK;
}

// Allocates `pages` pages: the first free run that is long enough, else the
// longest free runs until the request is met. false if the pool is short.
bool alloc_pages(pic_store *s, int64_t pages, std::vector<Run> &out) {
  out.clear();
  for (auto it = s->free_runs.begin(); it != s->free_runs.end(); ++it) {
    if (it->second < pages) continue;
    out.push_back(Run{it->first, (int32_t)pages, 0, 0});
    const int64_t rest = it->second - pages, start = it->first + pages;
    s->free_runs.erase(it);
    if (rest > 0) s->free_runs.emplace(start, rest);
    return true;
  }
  int64_t total = 0;
  for (auto &fr : s->free_runs) total += fr.second;
  if (total < pages) return false;
  std::vector<std::pair<int64_t, int64_t>> runs(s->free_runs.begin(), s->free_runs.end());
  std::stable_sort(runs.begin(), runs.end(),
                   [](const std::pair<int64_t, int64_t> &a, const std::pair<int64_t, int64_t> &b) {
                     return a.second > b.second;
                   });
  int64_t need = pages;
  for (auto &r : runs) {
    const int64_t take = std::min(need, r.second);
    out.push_back(Run{r.first, (int32_t)take, 0, 0});
    s->free_runs.erase(r.first);
    if (take < r.second) s->free_runs.emplace(r.first + take, r.second - take);
    need -= take;
    if (need == 0) break;
  }
  std::sort(out.begin(), out.end(), [](const Run &a, const Run &b) { return a.page0 < b.page0; });
  return true;
}

// Link-table entry of one run of a chunk in `layer`.
LinkEntry run_entry(const pic_store *s, const Run &r, int32_t layer) {
  const int64_t slot_tok_bytes = (s->k_tok_elems + s->v_tok_elems) * s->esz;
  const int32_t lp = r.pages * kTile;
  const int64_t skip_tok = (int64_t)r.skip * kTile;
  const char *block = s->pool + (int64_t)layer * s->layer_bytes + r.page0 * kTile * slot_tok_bytes;
  LinkEntry E{};
  // K rows and V^T panels of the view start skip_tok tokens into the block
  // (skip_tok is a multiple of the 32-token panel: skip_tok * d_v elements)
  E.k = block + skip_tok * s->desc.d_k * s->esz;
  E.v = s->desc.kind == PIC_GQA
            ? block + (int64_t)lp * s->k_tok_elems * s->esz + skip_tok * s->desc.d_v * s->esz
            : E.k;
  E.len = r.ntok;
  E.lp = lp;
  return E;
}

// Pages for a new chunk: free ones, else those of removed chunks whose
// readers are done, else after waiting for the remaining readers.
pic_status take_pages(pic_store *s, int64_t pages, std::vector<Run> &runs) {
  runs.clear();
  if (pages == 0) return PIC_OK;
  pic_status rc = reclaim(s, false);
  if (rc != PIC_OK) return rc;
  if (!alloc_pages(s, pages, runs) && !s->pending.empty()) {
    rc = reclaim(s, true);
    if (rc != PIC_OK) return rc;
    (void)alloc_pages(s, pages, runs);
  }
  if (runs.empty())
    return fail(PIC_ERR_OOM, "pool full: %lld of %lld tokens in use, %lld needed",
                (long long)s->used, (long long)s->capacity, (long long)pages * kTile);
  return PIC_OK;
}

// Host row list of pic_store_derive / pic_store_write_rows: strictly
// increasing, each below len.
bool check_rows(const int32_t *rows, int32_t n, int64_t len) {
  if (n < 0 || (n > 0 && !rows)) return false;
  for (int32_t i = 0; i < n; ++i)
    if (rows[i] < 0 || rows[i] >= len || (i > 0 && rows[i] <= rows[i - 1])) return false;
  return true;
}

// Adds d to the reference count of every page a chunk's views cover.
void ref_pages(pic_store *s, const std::vector<Run> &views, int32_t d) {
  for (const Run &v : views) {
    const int64_t first = v.page0 + v.skip, n = (v.ntok + kTile - 1) / kTile;
    for (int64_t p = first; p < first + n; ++p) s->page_refs[p] += d;
  }
}

// The view of a chunk holding token t.
const Run &view_of(const Slot &sl, int64_t t) {
  size_t i = 0;
  while (i + 1 < sl.runs.size() && sl.runs[i].tok0 + sl.runs[i].ntok <= t) ++i;
  return sl.runs[i];
}

bool check_offsets(const int32_t *a, int32_t n) {
  if (!a || a[0] != 0) return false;
  for (int32_t i = 0; i < n; ++i)
    if (a[i + 1] < a[i]) return false;
  return true;
}

// Validated, resolved form of one link call.
struct Plan {
  std::vector<LinkEntry> links;  // per request: its document links, then its own KV
  std::vector<ReqEntry> reqs;
  std::vector<int32_t> order;
  std::vector<std::pair<int32_t, int64_t>> own;   // (link index, workspace byte offset)
  int64_t own_bytes = 0;
  int32_t max_own_lp = 0;
  int32_t total_q = 0;
  int32_t max_rows = 0;          // max over requests of lq * group
  int32_t max_tiles = 0;
  bool self = false;             // requests carry own KV
  int64_t total_self = 0;        // own tokens over the batch
  std::vector<uint64_t> ids;     // every linked chunk id (with repeats)
  // per query token: linked rows visible to it; empty unless the rows of
  // some request see different numbers of them (the kernels mask per row)
  std::vector<int32_t> doc_lim;
};

// Tensor arguments of a call against its plan.
pic_status check_tensors(const pic_store *s, const Plan &P, const void *q, const void *k_self,
                         const void *v_self, const void *out) {
  if (P.total_q > 0 && (!q || !out)) return fail(PIC_ERR_INVALID, "q/out is NULL");
  if (P.self) {
    if (P.total_self > 0 && !k_self) return fail(PIC_ERR_INVALID, "k_self is NULL");
    if (s->desc.kind == PIC_GQA && P.total_self > 0 && !v_self)
      return fail(PIC_ERR_INVALID, "v_self is NULL");
    if (s->desc.kind == PIC_MLA && v_self) return fail(PIC_ERR_INVALID, "v_self must be NULL for MLA");
  } else if (k_self || v_self) {
    return fail(PIC_ERR_INVALID, "k_self/v_self given without self_offsets");
  }
  return PIC_OK;
}

// Validates a request batch and resolves its chunk ids into the link and
// request tables, with chunk addresses in cross-attention layer `layer`.
pic_status plan_call(pic_store *s, const pic_link_req *req, int32_t n_q_heads, float scale,
                     int32_t layer, int32_t max_q_per_req, Plan &P) {
  if (!s) return fail(PIC_ERR_INVALID, "store is NULL");
  if (!req) return fail(PIC_ERR_INVALID, "req is NULL");
  if (layer < 0 || layer >= s->n_layers)
    return fail(PIC_ERR_INVALID, "layer %d outside the store's %d layers", layer, s->n_layers);
  const pic_store_desc &d = s->desc;
  const int32_t B = req->batch;
  if (B < 0) return fail(PIC_ERR_INVALID, "batch < 0");
  if (n_q_heads <= 0 || n_q_heads % d.n_kv_heads)
    return fail(PIC_ERR_INVALID, "n_q_heads (%d) must be a positive multiple of n_kv_heads (%d)",
                n_q_heads, d.n_kv_heads);
  if (!std::isfinite(scale) || !(scale > 0.f))
    return fail(PIC_ERR_INVALID, "softmax_scale must be positive and finite");
  if (B == 0) return PIC_OK;
  if (!check_offsets(req->chunk_offsets, B)) return fail(PIC_ERR_INVALID, "bad chunk_offsets");
  if (!check_offsets(req->q_offsets, B)) return fail(PIC_ERR_INVALID, "bad q_offsets");
  const bool self = req->self_offsets != nullptr;
  if (self && !check_offsets(req->self_offsets, B)) return fail(PIC_ERR_INVALID, "bad self_offsets");
  const int64_t n_links = req->chunk_offsets[B];
  const int64_t tq = req->q_offsets[B];
  const int64_t ts = self ? req->self_offsets[B] : 0;
  if (n_links > 0 && !req->chunk_ids) return fail(PIC_ERR_INVALID, "chunk_ids is NULL");
  if (tq * n_q_heads > INT32_MAX / 2) return fail(PIC_ERR_INVALID, "too many query rows");
  P.self = self;
  P.total_self = ts;
  const int group = n_q_heads / d.n_kv_heads;
  const int64_t slot_tok_bytes = (s->k_tok_elems + s->v_tok_elems) * s->esz;
  P.links.clear();
  P.links.reserve(n_links + B);
  P.ids.clear();
  P.reqs.resize(B);
  P.doc_lim.clear();
  bool mixed_limits = false;
  std::vector<int64_t> weight(B);
  for (int32_t r = 0; r < B; ++r) {
    ReqEntry &R = P.reqs[r];
    const int32_t c0 = req->chunk_offsets[r], nc = req->chunk_offsets[r + 1] - c0;
    R.link0 = (int32_t)P.links.size();
    R.q0 = req->q_offsets[r];
    R.lq = req->q_offsets[r + 1] - R.q0;
    R.s0 = self ? req->self_offsets[r] : 0;
    R.ls = self ? req->self_offsets[r + 1] - R.s0 : 0;
    if (self && R.ls < R.lq)
      return fail(PIC_ERR_INVALID, "request %d: %d query tokens but only %d own tokens", r, R.lq,
                  R.ls);
    if (R.lq > max_q_per_req)
      return fail(PIC_ERR_INVALID, "request %d: %d query tokens exceeds %d", r, R.lq,
                  max_q_per_req);
    int64_t tiles = 0, toks = 0;
    for (int32_t c = 0; c < nc; ++c) {
      const uint64_t id = req->chunk_ids[c0 + c];
      auto it = s->map.find(id);
      if (it == s->map.end())
        return fail(PIC_ERR_NOT_FOUND, "request %d link %d: chunk id 0x%llx not in the store", r,
                    c, (unsigned long long)id);
      const Slot &sl = it->second;
      const int32_t start = req->chunk_starts ? req->chunk_starts[c0 + c] : 0;
      if (start < 0 || start % kTile || start >= sl.len)
        return fail(PIC_ERR_INVALID,
                    "request %d link %d: start %d must be a multiple of %d below the chunk's %lld "
                    "tokens", r, c, start, kTile, (long long)sl.len);
      for (const Run &run : sl.runs) {
        if (run.tok0 + run.ntok <= start) continue;
        LinkEntry E = run_entry(s, run, layer);
        // skip the run's pages before `start`: rows of K, panels of V^T
        // (the head stride stays the run's)
        const int32_t skip = std::max(0, start - run.tok0);
        E.k = (const char *)E.k + (int64_t)skip * d.d_k * s->esz;
        E.v = d.kind == PIC_MLA ? E.k : (const char *)E.v + (int64_t)skip * d.d_v * s->esz;
        E.len -= skip;
        E.tile0 = (int32_t)tiles;
        E.tok0 = (int32_t)toks;
        P.links.push_back(E);
        tiles += (E.len + kTile - 1) / kTile;
        toks += E.len;
      }
      P.ids.push_back(id);
    }
    if (req->q_doc_limits && R.lq > 0) {
      int32_t lo = INT32_MAX, hi = 0;
      for (int32_t i = 0; i < R.lq; ++i) {
        const int32_t lim = req->q_doc_limits[R.q0 + i];
        if (lim < 0 || lim > toks)
          return fail(PIC_ERR_INVALID, "request %d query %d: limit %d outside 0..%lld linked rows",
                      r, i, lim, (long long)toks);
        lo = std::min(lo, lim);
        hi = std::max(hi, lim);
      }
      // rows past every query's limit are never read: cut the links there;
      // limits that differ between rows are applied by the kernels
      if (hi < toks) {
        size_t keep = R.link0;
        tiles = 0;
        while (keep < P.links.size() && P.links[keep].tok0 < hi) {
          LinkEntry &E = P.links[keep++];
          E.len = std::min(E.len, hi - E.tok0);
          tiles += (E.len + kTile - 1) / kTile;
        }
        P.links.resize(keep);
        toks = hi;
      }
      if (lo < hi) mixed_limits = true;
    }
    if (toks + R.ls > INT32_MAX / 2) return fail(PIC_ERR_INVALID, "request %d too long", r);
    R.doc_tiles = (int32_t)tiles;
    if (R.ls > 0) {             // own KV: a slot in the call's workspace, filled on the device
      LinkEntry E{};
      E.len = R.ls;
      E.lp = (int32_t)round_up(R.ls, kTile);
      E.tile0 = (int32_t)tiles;
      E.tok0 = (int32_t)toks;
      P.own.emplace_back((int32_t)P.links.size(), P.own_bytes);
      P.own_bytes += round_up((int64_t)E.lp * slot_tok_bytes, 256);
      P.max_own_lp = std::max(P.max_own_lp, E.lp);
      P.links.push_back(E);
      tiles += E.lp / kTile;
    }
    R.nlinks = (int32_t)P.links.size() - R.link0;
    R.tiles = (int32_t)tiles;
    P.max_rows = std::max(P.max_rows, R.lq * group);
    P.max_tiles = std::max(P.max_tiles, R.tiles);
    weight[r] = (int64_t)R.tiles * R.lq;
  }
  P.order.resize(B);
  for (int32_t r = 0; r < B; ++r) P.order[r] = r;
  std::stable_sort(P.order.begin(), P.order.end(),
                   [&](int32_t a, int32_t b) { return weight[a] > weight[b]; });
  P.total_q = (int32_t)tq;
  if (mixed_limits) P.doc_lim.assign(req->q_doc_limits, req->q_doc_limits + tq);
  return PIC_OK;
}

// Points the own-KV links of `links` (the plan's tables) at their slots in
// the workspace `work`.
void place_own(const pic_store *s, const Plan &P, void *work, LinkEntry *links) {
  const bool mla = s->desc.kind == PIC_MLA;
  for (auto &o : P.own) {
    LinkEntry &E = links[o.first];
    E.k = (char *)work + o.second;
    E.v = mla ? E.k : (const char *)E.k + (int64_t)E.lp * s->k_tok_elems * s->esz;
  }
}

// Where the prologue reads the tables, and what it copies first.
struct Prologue {
  const LinkEntry *links = nullptr;
  const ReqEntry *reqs = nullptr;
  const void *copy_src = nullptr;
  void *copy_dst = nullptr;
  int64_t copy_bytes = 0;
};

void prof_start(hipStream_t st, std::pair<hipEvent_t, hipEvent_t> *ev) {
  ev->first = ev->second = nullptr;
  std::lock_guard<std::mutex> g(g_prof.mu);
  if (!g_prof.on) return;
  if (g_prof.seen++ % g_prof.every) return;
  if (!g_prof.spare.empty()) {
    *ev = g_prof.spare.back();
    g_prof.spare.pop_back();
  } else if (hipEventCreateWithFlags(&ev->first, hipEventDisableSystemFence) != hipSuccess ||
             hipEventCreateWithFlags(&ev->second, hipEventDisableSystemFence) != hipSuccess) {
    // timing-only events: a system-scope fence would add a cache writeback
    // and invalidation around the timed kernel
    ev->first = ev->second = nullptr;
    return;
  }
  (void)hipEventRecord(ev->first, st);
}

void prof_stop(hipStream_t st, std::pair<hipEvent_t, hipEvent_t> *ev, const char *name) {
  if (!ev->first) return;
  (void)hipEventRecord(ev->second, st);
  std::lock_guard<std::mutex> g(g_prof.mu);
  g_prof.events.push_back(*ev);
  g_prof.name = name;
}

enum class Mode { Prefill, Decode };
enum class Kern { Valu, Mfma128, Decode128, Mla, Stream };

// Everything about a call that does not depend on its tensors: the resolved
// tables, the kernel, the split count and the workspace layout
// [own KV slots, laid out like chunk slots][split partials].
struct Setup {
  Plan P;
  Kern kern = Kern::Valu;
  int32_t splits = 1;            // most pieces of a request
  std::vector<int32_t> req_splits;   // pieces per request (kernels that take work items)
  std::vector<CombineEntry> comb;    // their partial rows (when some request is split)
  int32_t tile_keys = kTile;     // keys per tile of the kernel's work items
  int32_t n_items = 0;
  bool lean = false;             // a small call the lean kernel runs
  bool small = false;            // tables as a kernel argument, own KV in place
  int32_t rows_per_block = 0;    // rows of a workgroup (decode kernel: wave)
  int32_t stream_rows = 0;       // stream kernel: rows per wave
  LinkParams lp{};               // shapes only: no tables, tensors or scale yet
  std::vector<OwnArg> own_args;  // per request, for the prologue (batch <= kOwnArgs)
  int64_t part_rows = 0;         // partial rows of the call
  size_t part_off = 0, part_bytes = 0;
  size_t work_bytes() const { return part_off + part_bytes; }
};

// Layout of a call's tables: links, requests, request order, per-query
// limits, work items, combine entries.
struct TableLayout {
  size_t off_r, off_o, off_d, off_i, off_c, bytes;
};
TableLayout table_layout(const Setup &C) {
  const size_t nl = C.P.links.size(), nr = C.P.reqs.size();
  TableLayout t;
  t.off_r = round_up(sizeof(LinkEntry) * nl, 256);
  t.off_o = t.off_r + round_up(sizeof(ReqEntry) * nr, 256);
  t.off_d = t.off_o + round_up(sizeof(int32_t) * nr, 256);
  t.off_i = t.off_d + round_up(sizeof(int32_t) * C.P.doc_lim.size(), 256);
  t.off_c = t.off_i + round_up(sizeof(WorkItem) * C.n_items, 256);
  t.bytes = t.off_c + round_up(sizeof(CombineEntry) * C.comb.size(), 256);
  return t;
}

// The call's work items in dispatch order: C.P.order's requests, each one's
// pieces in key order. links: the call's link table (own-KV links placed).
void write_items(const Setup &C, const LinkEntry *links, WorkItem *out) {
  const int per = kTile / C.tile_keys;     // kernel tiles per 64-key tile
  for (int32_t r : C.P.order) {
    const ReqEntry &R = C.P.reqs[r];
    const int64_t S = C.req_splits[r], tiles = (int64_t)R.tiles * per;
    int32_t li = R.link0;
    for (int64_t i = 0; i < S; ++i) {
      WorkItem w{};
      w.t_begin = (int32_t)(tiles * i / S);
      w.t_end = (int32_t)(tiles * (i + 1) / S);
      if (w.t_begin < w.t_end) {
        while (li + 1 < R.link0 + R.nlinks && links[li + 1].tile0 * per <= w.t_begin) ++li;
        const LinkEntry &L = links[li];
        w.k = L.k;
        w.v = L.v;
        w.len = L.len;
        w.lp = L.lp;
        w.tile0 = L.tile0;
        w.tok0 = L.tok0;
      }
      if (C.kern == Kern::Decode128) w.tok0 = R.s0;   // it masks no linked rows
      w.link = li;
      w.q0 = R.q0;
      w.lq = R.lq;
      w.ls = R.ls;
      w.doc_tiles = R.doc_tiles;
      w.part = S > 1 ? (int32_t)(C.comb[r].part0 + i * C.comb[r].rows) : -1;
      *out++ = w;
    }
  }
}

// Writes the call's tables (host memory, laid out by t) for one layer's
// links.
void write_tables(const Setup &C, const TableLayout &t, const LinkEntry *links, char *h) {
  const Plan &P = C.P;
  if (!P.links.empty()) memcpy(h, links, sizeof(LinkEntry) * P.links.size());
  if (!P.reqs.empty()) {
    memcpy(h + t.off_r, P.reqs.data(), sizeof(ReqEntry) * P.reqs.size());
    memcpy(h + t.off_o, P.order.data(), sizeof(int32_t) * P.reqs.size());
  }
  if (!P.doc_lim.empty())
    memcpy(h + t.off_d, P.doc_lim.data(), sizeof(int32_t) * P.doc_lim.size());
  if (C.n_items > 0) write_items(C, links, (WorkItem *)(h + t.off_i));
  if (!C.comb.empty())
    memcpy(h + t.off_c, C.comb.data(), sizeof(CombineEntry) * C.comb.size());
}

// Points lp's tables at their device copy.
void point_tables(const Setup &C, const TableLayout &t, const char *dev, LinkParams &lp) {
  lp.links = (const LinkEntry *)dev;
  lp.reqs = (const ReqEntry *)(dev + t.off_r);
  lp.order = (const int32_t *)(dev + t.off_o);
  lp.doc_lim = C.P.doc_lim.empty() ? nullptr : (const int32_t *)(dev + t.off_d);
  lp.items = C.n_items > 0 ? (const WorkItem *)(dev + t.off_i) : nullptr;
  lp.comb = C.comb.empty() ? nullptr : (const CombineEntry *)(dev + t.off_c);
}

// Writes the call's tables into a staging slot (host-mapped pinned memory)
// and points lp's tables at the slot's device copy; the call's prologue
// kernel moves them there. The slot also holds the call's workspace, where
// the own-KV links are pointed.
pic_status upload(pic_store *s, Setup &C, Stage **stage, LinkParams &lp, TableLayout &tl) {
  tl = table_layout(C);
  pic_status rc = stage_acquire(s, tl.bytes, stage);
  if (rc != PIC_OK) return rc;
  if (C.work_bytes() > 0) {
    rc = ensure_work(*stage, C.work_bytes());
    if (rc != PIC_OK) return rc;
  }
  place_own(s, C.P, (*stage)->work, C.P.links.data());
  write_tables(C, tl, C.P.links.data(), (char *)(*stage)->host);
  point_tables(C, tl, (const char *)(*stage)->dev, lp);
  return PIC_OK;
}

// What a kernel's pieces cost, in its tiles.
struct SplitCost {
  int64_t slots;       // workgroups (decode kernel: waves) the GPU holds at once
  int64_t fit;         // ... that a round is planned with
  double over;         // a piece's fixed time: start, first loads, epilogue
  double part;         // writing and merging one partial row
  double fixed;        // the combine launch
  int32_t min_piece;   // fewest tiles of a piece
  bool lockstep;       // see choose_splits
  int32_t max_splits;
};

// Pieces per request, so that the call finishes early: candidate piece
// lengths L are the shortest for which the call's workgroups still fit half,
// one, two, three or four rounds of the GPU, and the whole request; each
// costs its longest piece if the workgroups all run at once, else the
// average work per slot plus 0.3 of the longest piece (in-order dispatch
// leaves the last pieces uneven), and in both cases the partials its splits
// write and merge. lockstep: like pieces of the fp32 128-wide stream kernel,
// one workgroup per CU bound by its matrix instructions, start and end
// together, so a call takes a shortest piece for every round begun, and up to
// eight rounds of short pieces are considered (9 requests of 300 tokens x 24/8
// heads over 6 links of 1024: unsplit, 2.25 rounds, 2475 us, in 3 pieces 2030).
// Requests are cut into equal pieces of at most L tiles, so
// a ragged batch gets pieces of like length (with one split count for all
// requests the longest request's pieces set the time: an MLA decode step of
// 32 requests over 4..14 links took 58 us in 8 pieces each).
// tiles, blocks, rows: per request its key tiles, its workgroups per piece
// and its output rows. share: the mean part of its tiles that its row blocks
// walk (below 1 with per-query limits; pieces past a block's part are empty
// and cost next to nothing), so S pieces are share x S + 1 - share workgroups
// per row block.
std::vector<int32_t> choose_splits(const std::vector<int32_t> &tiles,
                                   const std::vector<int32_t> &blocks,
                                   const std::vector<int64_t> &rows,
                                   const std::vector<double> &share, const SplitCost &c) {
  const size_t n = tiles.size();
  // ceil(tiles / L); + 0.5 keeps the product off the integers it is cut at
  auto pieces = [&](size_t r, int32_t L, double inv) {
    const int32_t s = (int32_t)((tiles[r] + L - 1 + 0.5) * inv);
    return std::min(c.max_splits, std::max(1, s));
  };
  auto total = [&](int32_t L) {
    const double inv = 1.0 / L;
    double t = 0;
    for (size_t r = 0; r < n; ++r)
      t += blocks[r] * (pieces(r, L, inv) * share[r] + 1 - share[r]);
    return t;
  };
  auto cost = [&](int32_t L) {
    const double inv = 1.0 / L;
    double work = 0, longest = 0, shortest = 1e30, part = 0, wgs = 0;
    for (size_t r = 0; r < n; ++r) {
      if (blocks[r] == 0) continue;
      const int32_t S = pieces(r, L, inv);
      const double held = blocks[r] * (S * share[r] + 1 - share[r]);
      wgs += held;
      work += blocks[r] * tiles[r] * share[r] + c.over * held;
      longest = std::max(longest, (double)((tiles[r] + S - 1) / S) + c.over);
      shortest = std::min(shortest, (double)(tiles[r] / S) + c.over);
      if (S > 1) part += c.part * (double)rows[r] * S * share[r];
    }
    double run = longest;
    if (c.lockstep)
      run = std::max({longest, work / (double)c.slots + 0.3 * (longest - shortest),
                      std::ceil(wgs / (double)c.slots) * shortest});
    else if (wgs > (double)c.slots)
      run = std::max(longest, work / (double)c.slots + 0.3 * longest);
    return run + part + (part > 0 ? c.fixed : 0.0);
  };
  int32_t most = 1;
  for (size_t r = 0; r < n; ++r) most = std::max(most, tiles[r]);
  int32_t best_L = most;
  double best = cost(most);
  for (int k : {1, 2, 4, 6, 8, 10, 12, 14, 16}) {          // half rounds
    if (k > 8 && !c.lockstep) break;
    const double limit = (double)(c.fit * k / 2);
    if (total(most) > limit) continue;
    int32_t lo = std::min(c.min_piece, most), hi = most;   // shortest L that fits
    while (lo < hi) {
      const int32_t mid = (lo + hi) / 2;
      if (total(mid) <= limit)
        hi = mid;
      else
        lo = mid + 1;
    }
    const double t = cost(lo);
    if (t < best) {
      best = t;
      best_L = lo;
    }
  }
  std::vector<int32_t> S(n);
  for (size_t r = 0; r < n; ++r) S[r] = pieces(r, best_L, 1.0 / best_L);
  return S;
}

// Request order for the d128 prefill kernel. Workgroup j of XCD x runs row
// block j % nrb of group x + n_xcd (j / nrb) (see the kernel's work
// mapping) and starts on the first of the XCD's slots (CUs times workgroups
// per CU) that frees up, as the in-order dispatch does; with n_kv a multiple
// of n_xcd every XCD sees the same sequence of requests, each n_kv / n_xcd
// times. Heaviest first is the usual list-scheduling order; when an XCD's
// workgroups take several rounds of its slots, one pass of pairwise swaps
// that shorten the simulated finish time improves on it (long_rag: 957 ->
// 934 tiles, against a bound of 916). A workgroup takes its visible tiles
// plus 1.5 (its query rows, first tile and epilogue). The search keeps the
// slot times after each prefix of the order and stops a trial once some
// slot passes the best finish time; the result is kept for the next call
// with the same request shapes (a batch linked at every cross-attention
// layer or decode step). Other shapes keep heaviest first.
struct OrderSim {
  const Plan *P;
  int nrb, rows_per_block, group, reps, slots;
  double dur(int r, int rb) const {
    const ReqEntry &R = P->reqs[r];
    const int rows = R.lq * group, row0 = rb * rows_per_block;
    if (row0 >= rows) return -1.0;    // the workgroup returns at once
    return visible_tiles(R, std::min(rows - 1, row0 + rows_per_block - 1) / group) + 1.5;
  }
  // Adds request r's workgroups to the slot times `h` (a min-heap); false
  // once some slot passes `limit`.
  bool add(std::vector<double> &h, double &top, int r, double limit) const {
    for (int k = 0; k < reps; ++k)
      for (int rb = 0; rb < nrb; ++rb) {
        const double d = dur(r, rb);
        if (d < 0) continue;
        std::pop_heap(h.begin(), h.end(), std::greater<double>());
        h.back() += d;
        top = std::max(top, h.back());
        std::push_heap(h.begin(), h.end(), std::greater<double>());
        if (top >= limit) return false;
      }
    return true;
  }
};

// finish: when not NULL, receives the simulated finish time (in tiles) of
// the busiest XCD for heaviest first and for the order chosen (both 0 when
// no search runs). s: the store whose memo to use, or NULL for none.
void balance_order_d128(pic_store *s, Plan &P, const LinkParams &lp, int rows_per_block,
                        int slots, double *finish = nullptr) {
  if (finish) finish[0] = finish[1] = 0;
  const int B = (int)P.order.size();
  if (B < 3 || B > 64 || slots <= 0 || lp.n_kv_heads % lp.n_xcd) return;
  const int reps = lp.n_kv_heads / lp.n_xcd;
  if ((int64_t)B * reps * lp.nrb <= slots) return;   // one round: all start at once
  std::vector<int32_t> key = {lp.nrb, rows_per_block, lp.group, reps, slots, B};
  for (const ReqEntry &R : P.reqs) key.insert(key.end(), {R.lq, R.ls, R.doc_tiles, R.tiles});
  if (s && !finish && key == s->order_key) {
    P.order = s->order_memo;
    return;
  }
  const OrderSim sim{&P, lp.nrb, rows_per_block, lp.group, reps, slots};
  std::vector<int32_t> order = P.order;
  std::vector<double> pre(slots, 0.0), h;
  double pre_top = 0, best = 0;
  {
    h = pre;
    for (int i = 0; i < B; ++i) sim.add(h, best, order[i], INFINITY);
  }
  if (finish) finish[0] = best;
  auto same_shape = [&](int a, int b) {
    const ReqEntry &x = P.reqs[a], &y = P.reqs[b];
    return x.lq == y.lq && x.ls == y.ls && x.doc_tiles == y.doc_tiles && x.tiles == y.tiles;
  };
  for (int i = 0; i + 1 < B; ++i) {
    for (int j = i + 1; j < B; ++j) {
      if (same_shape(order[i], order[j])) continue;
      std::swap(order[i], order[j]);
      h = pre;
      double top = pre_top;
      bool ok = true;
      for (int k = i; k < B && ok; ++k) ok = sim.add(h, top, order[k], best - 1e-9);
      if (ok)
        best = top;
      else
        std::swap(order[i], order[j]);
    }
    sim.add(pre, pre_top, order[i], INFINITY);
  }
  if (finish) finish[1] = best;
  P.order = order;
  if (s) {
    s->order_key = std::move(key);
    s->order_memo = order;
  }
}

// Tables that travel as a kernel argument (SmallTabs): such a call of a
// kernel that reads its own-KV tiles from k_self / v_self skips the
// prologue. For latency-bound calls the prologue was a sixth of the step
// (tiny_f32: 3.7 of 23.4 us).
bool small_tables(const Plan &P) {
  return P.links.size() <= (size_t)kSmallLinks && P.reqs.size() <= (size_t)kSmallReqs &&
         P.doc_lim.empty();
}

// Most rows per kv head of a prefill call of the stream kernel that takes the
// small form (no prologue, but own values gathered by every row block and one
// split count for all requests). Small against other form, 24/8 heads, one
// request over 10 links of 512 unless said: bf16 x 64, 129 rows 20.3 against
// 25.2 us, 6 requests of 129 / 192 / 384 rows over 4 links 28.5 / 31.0 / 55.5
// against 31.7 / 34.9 / 45.3; fp32 x 64, 48 / 96 / 129 / 288 rows 28.5 / 37.8 /
// 40.5 / 60.7 against 29.7 / 32.5 / 42.7 / 56.2. Up to 128 rows bf16 always
// gains; fp32 gains or loses with how its split count falls.
constexpr int kStreamSmallRows = 128;

// Costs of a kernel's pieces in its tiles (see choose_splits). Tile times on
// a full GPU: d128 1.75 us per workgroup (64 keys), MLA 2.0 us (64 keys),
// decode 5 us per wave (32 keys, eight waves per CU on the HBM stream),
// stream kernel below. Partials move at about 4 TB/s, written and read; a
// combine launch is about 4.5 us.
// uneven_rows: some request has fewer row blocks than another.
SplitCost split_cost(Kern kern, int32_t cus, const pic_store_desc &d, int32_t max_rows,
                     const StreamShape &ss, bool uneven_rows) {
  const double part_us = (d.d_v + 2) * 8.0 / 4e6;
  SplitCost c{};
  c.max_splits = 256;
  double us = 1;
  if (kern == Kern::Mfma128) {
    us = 1.75;
    c.slots = (int64_t)cus * mfma_d128_blocks_per_cu();
    c.over = 3;
    // a piece reads more keys and values than the partials it writes and the
    // combine reads back
    const int64_t part = 2 * (int64_t)std::min(max_rows, mfma_d128_rows_per_block()) * (d.d_v + 2) * 4;
    const int64_t tile = (int64_t)kTile * (d.d_k + d.d_v) * 2;
    c.min_piece = (int32_t)std::max<int64_t>(1, std::min<int64_t>(8, part / tile));
  } else if (kern == Kern::Mla) {
    us = 2.0;
    c.slots = cus;
    c.over = 4;
    c.min_piece = 2;
  } else if (kern == Kern::Decode128) {
    us = 5.0;
    c.slots = 8 * (int64_t)cus;
    c.over = 2;
    c.min_piece = 1;
  } else {
    // Cycles of a wave's 32-key tile. fp32: D / 16 x 16 matrix instructions of
    // 32 cycles per 16 rows. bf16: 22 per row. Measured, 8 requests x 512 tokens
    // x 32/8 heads over 16 links of 1024, two workgroups per CU: 1.65 us per
    // tile for bf16 x 64 (28 cycles per row at 2.2 GHz), 1.32 for bf16 x 32
    // (22), 4.15 for fp32 x 64, and 4.24 for fp32 x 128, one workgroup per CU.
    // The waves of a workgroup share a tile kpar ways.
    const double cyc = d.dtype == PIC_F32 ? 2.0 * d.d_k * ss.rows : 22.0 * ss.rows;
    // Requests with different numbers of row blocks fill the CUs unevenly; with
    // one workgroup per CU they are planned as for two, in finer pieces than
    // the rounds ask for (12 requests of 20..130 tokens over 6 links of 700,
    // 32/8, 24/8 and 6/2 heads: 737, 543 and 176 us, planned for one 772, 594
    // and 191).
    c.lockstep = ss.per_cu == 1 && !uneven_rows;
    const int wgs = c.lockstep ? 1 : 2;
    us = wgs * cyc / 2200.0 / ss.kpar;
    c.slots = wgs * (int64_t)cus;
    c.over = 6.0 / us;
    c.min_piece = 2 * ss.kpar;
  }
  // Where requests have different numbers of row blocks, the empty ones leave
  // the XCDs and CUs unevenly filled, and a round planned full runs over on
  // some of them: an eighth stays free (12 fp32 requests of 20..130 tokens:
  // 77 us with a twentieth free, 64 us with a tenth or more; 8 bf16 requests
  // of 30..300 tokens, 64-wide heads: 168 us full, 147 us).
  c.fit = uneven_rows ? c.slots * 7 / 8 : c.slots;
  c.part = part_us / us;
  c.fixed = 4.5 / us;
  return c;
}

// Mean over a request's row blocks of the share of its linked rows that lie
// below the farthest limit of the block's query tokens.
double limit_share(const Plan &P, const ReqEntry &R, int group, int rows_per_block, int64_t linked) {
  const int64_t rows = (int64_t)R.lq * group;
  double sum = 0;
  int n = 0;
  for (int64_t row0 = 0; row0 < rows; row0 += rows_per_block, ++n) {
    const int64_t last = std::min(rows, row0 + rows_per_block) - 1;
    int32_t far = 0;
    for (int64_t t = row0 / group; t <= last / group; ++t) far = std::max(far, P.doc_lim[R.q0 + t]);
    sum += linked > 0 ? (double)far / (double)linked : 0.0;
  }
  return n ? sum / n : 1.0;
}

// Completes a call of work items from its pieces per request (C.req_splits):
// item counts, partial rows, request order, workspace layout.
void apply_splits(pic_store *s, int32_t n_q_heads, int rows_per_block, Setup &C) {
  Plan &P = C.P;
  LinkParams &lp = C.lp;
  const int B = (int)P.reqs.size();
  C.n_items = 0;
  C.splits = 1;
  lp.even = 1;
  for (int r = 0; r < B; ++r) {
    if (P.reqs[r].lq == 0) C.req_splits[r] = 1;
    C.n_items += C.req_splits[r];
    C.splits = std::max(C.splits, C.req_splits[r]);
    if (P.reqs[r].tiles != P.reqs[0].tiles || P.reqs[r].lq != P.reqs[0].lq) lp.even = 0;
  }
  lp.n_items = C.n_items;
  lp.num_splits = C.splits;
  lp.gang = std::max(1, s->shape.cus / s->shape.xcds);
  // The stream kernel always spreads the row blocks of a unit over the XCDs:
  // its row blocks are short and many, and ragged batches leave XCDs idle
  // otherwise (12 requests of 20..130 tokens, 24/8 heads, over 6 links of 700:
  // fp32 x 64 279 us, by the rule 451; bf16 x 64 92, 124; bf16 x 32 77, 99; even
  // batches of 256 and 512 tokens within 2% of each other).
  lp.spread = C.kern == Kern::Stream ||
              spread_units((int64_t)C.n_items * lp.n_kv_heads, lp.nrb, lp.n_xcd);
  // With per-query limits the early row blocks of late pieces are empty: the
  // last row blocks start first, the empty ones fill in at the end (dispatched
  // among the others, they delayed the start of some: S = 4 pieces 54 us, 3
  // pieces 43 us).
  if (C.kern == Kern::Mfma128 && lp.skip_empty && lp.nrb > 1) lp.spread = 2;
  C.part_rows = 0;
  C.comb.clear();
  if (C.splits > 1) {
    C.comb.resize(B);
    for (int r = 0; r < B; ++r) {
      const int32_t S = C.req_splits[r], rows = P.reqs[r].lq * n_q_heads;
      C.comb[r] = CombineEntry{P.reqs[r].q0 * n_q_heads, rows, (int32_t)C.part_rows, S};
      if (S > 1) C.part_rows += (int64_t)rows * S;
    }
    // longest pieces first
    std::stable_sort(P.order.begin(), P.order.end(), [&](int32_t a, int32_t b) {
      return (int64_t)P.reqs[a].tiles * C.req_splits[b] > (int64_t)P.reqs[b].tiles * C.req_splits[a];
    });
  } else if (C.kern == Kern::Mfma128 && !lp.spread) {
    balance_order_d128(s, P, lp, rows_per_block,
                       s->shape.cus / s->shape.xcds * mfma_d128_blocks_per_cu());
  }
  // The decode kernel reads the own KV in place: nothing to lay out.
  if (C.kern == Kern::Decode128) P.max_own_lp = 0;
  C.part_off = C.kern == Kern::Decode128 ? 0 : round_up(P.own_bytes, 256);
  C.part_bytes = (size_t)C.part_rows * (s->desc.d_v + 2) * sizeof(float);
}

// Most bytes of split partials the library's own choice of pieces may take.
// Four rounds of workgroups, the most choose_splits plans, write 4 x CUs x
// workgroups per CU x rows x (d_v + 2) fp32: 130 MiB for the d128 kernel, 128
// MLA, 132 for narrow bf16 heads, less for the others. Only calls with
// per-query limits reach the bound: the row blocks that walk next to nothing
// of a piece cost no time, so they are not counted as workgroups, but a piece
// has room for the partial rows of all of them (4096 query tokens x 32 heads
// that see one linked row of 65,536, but for the last: 32 pieces, 2.2 GB).
constexpr size_t kMostPartBytes = size_t(144) << 20;

// Cuts the pieces of the requests that have the most, by at least an eighth.
void fewer_pieces(pic_store *s, int32_t n_q_heads, Setup &C) {
  const int32_t most = C.splits - (C.splits + 7) / 8;
  for (int32_t &S : C.req_splits) S = std::min(S, most);
  apply_splits(s, n_q_heads, C.rows_per_block, C);
}

// Bytes of static scratch a pic_link_decode_noalloc call is charged for (its
// limit, stated in pic.h): tables, the own KV laid out, and partials of one
// split count for all requests, num_splits or, for 0, the one that gives
// about eight workgroups (decode kernel: waves) per CU, of 256 rows (d128),
// 64 (MLA) or 16 (others).
size_t noalloc_charge(const pic_store *s, const Setup &C, int32_t num_splits) {
  const Plan &P = C.P;
  const pic_store_desc &d = s->desc;
  const int block = C.kern == Kern::Mfma128 ? mfma_d128_rows_per_block()
                    : C.kern == Kern::Mla   ? mla_rows_per_block()
                                            : 16;
  int64_t splits = num_splits;
  if (splits == 0) {
    const int64_t blocks = (int64_t)P.reqs.size() * d.n_kv_heads *
                           std::max(1, (P.max_rows + block - 1) / block);
    splits = std::max<int64_t>(
        1, std::min<int64_t>((8 * (int64_t)s->shape.cus + blocks - 1) / blocks, 256));
    splits = std::min<int64_t>(splits, std::max(1, P.max_tiles));
  }
  const size_t part = splits > 1 ? (size_t)P.total_q * C.lp.n_q_heads * splits * (d.d_v + 2) * 4 : 0;
  if ((C.kern == Kern::Valu || C.kern == Kern::Stream) && small_tables(P)) return part;
  return round_up(sizeof(LinkEntry) * P.links.size(), 256) +
         round_up(sizeof(ReqEntry) * P.reqs.size(), 256) +
         round_up(sizeof(int32_t) * P.reqs.size(), 256) +
         round_up(sizeof(int32_t) * P.doc_lim.size(), 256) + round_up(P.own_bytes, 256) + part;
}

pic_status setup_call(pic_store *s, const pic_link_req *req, int32_t n_q_heads, float scale,
                      int32_t layer, int32_t num_splits, Mode mode, Setup &C) {
  if (mode == Mode::Decode && (num_splits < 0 || num_splits > 256))
    return fail(PIC_ERR_INVALID, "num_splits must be 0..256");
  Plan &P = C.P;
  pic_status rc = plan_call(s, req, n_q_heads, scale, layer,
                            mode == Mode::Decode ? 16 : INT32_MAX, P);
  if (rc != PIC_OK) return rc;
  const pic_store_desc &d = s->desc;
  const bool mla = d.kind == PIC_MLA;
  LinkParams &lp = C.lp;
  lp.batch = req->batch;
  lp.n_q_heads = n_q_heads;
  lp.n_kv_heads = d.n_kv_heads;
  lp.group = n_q_heads / d.n_kv_heads;
  lp.d_k = d.d_k;
  lp.d_v = d.d_v;
  lp.total_q = P.total_q;
  if (req->batch == 0 || P.total_q == 0) return PIC_OK;
  if (P.max_own_lp > 0 && req->batch <= kOwnArgs) {
    C.own_args.assign(req->batch, OwnArg{0, 0, 0});
    size_t k = 0;
    for (int32_t r = 0; r < req->batch; ++r) {
      const ReqEntry &R = P.reqs[r];
      if (R.ls == 0) continue;
      C.own_args[r] = OwnArg{R.s0, R.ls, P.own[k++].second};
    }
  }

  // Kernel choice.
  //   bf16 GQA d=128: decode-shaped calls with at most 16 rows per (request,
  //   kv head) stream keys with the decode kernel; everything else runs the
  //   matrix-core flash kernel (split when decoding).
  //   Other shapes / fp32 / MLA: the generic vector-ALU kernel.
  //   bf16 MLA with 576-wide latent rows and 512-wide values: the MLA
  //   matrix-core kernel (split when decoding).
  Kern kern = Kern::Valu;
  const bool bf16_128 = d.dtype == PIC_BF16 && !mla && d.d_k == 128 && d.d_v == 128;
  if (bf16_128)
    kern = mode == Mode::Decode && P.max_rows <= decode_d128_max_rows() ? Kern::Decode128
                                                                         : Kern::Mfma128;
  // rows of one request that see different numbers of linked rows need the
  // per-row masks of the flash kernel
  if (kern == Kern::Decode128 && !P.doc_lim.empty()) kern = Kern::Mfma128;
  if (d.dtype == PIC_BF16 && mla && d.d_k == 576 && d.d_v == 512) kern = Kern::Mla;
  // A small generic call of a shape the lean kernel is built for (tables as
  // a kernel argument, at most kLeanTiles tiles in all) runs it; other fp32
  // and narrow bf16 GQA calls stream their keys through the matrix cores.
  if (kern == Kern::Valu && !mla) {
    if (lean_supported(d.dtype, d.d_k, d.d_v, lp.group) && small_tables(P)) {
      int64_t tiles = 0;
      for (const ReqEntry &R : P.reqs) tiles += R.tiles;
      C.lean = tiles <= kLeanTiles;
    }
    if (!C.lean && stream_supported(d.dtype, d.d_k, d.d_v)) kern = Kern::Stream;
  }
  C.small = small_tables(P) &&
            (kern == Kern::Valu || (kern == Kern::Stream && (mode == Mode::Decode ||
                                                             P.max_rows <= kStreamSmallRows)));
  if (kern == Kern::Valu && valu_lds_bytes_for(s->esz, mla, d.d_k, d.d_v) > 160 * 1024)
    return fail(PIC_ERR_UNSUPPORTED, "head widths d_k=%d d_v=%d exceed the generic kernel's LDS",
                d.d_k, d.d_v);
  C.kern = kern;
  StreamShape ss{0, 1, 4};
  if (kern == Kern::Stream) ss = stream_shape(d.dtype, d.d_k, P.max_rows, C.small);
  lp.kpar = ss.kpar;
  C.stream_rows = ss.rows;
  const int rows_per_block = kern == Kern::Mfma128 ? mfma_d128_rows_per_block()
                             : kern == Kern::Stream ? ss.rows * 4 / ss.kpar
                             : kern == Kern::Valu  ? valu_rows_per_block()
                             : kern == Kern::Mla   ? mla_rows_per_block()
                                                   : decode_d128_max_rows();
  C.rows_per_block = rows_per_block;
  lp.nrb = std::max(1, (P.max_rows + rows_per_block - 1) / rows_per_block);
  lp.max_rows = P.max_rows;
  lp.n_groups = req->batch * d.n_kv_heads;
  lp.n_xcd = s->shape.xcds;

  const bool by_items = kern != Kern::Valu && !C.small;
  if (by_items) {
    C.tile_keys = kern == Kern::Decode128 || kern == Kern::Stream ? 32 : kTile;
    const int B = req->batch;
    std::vector<int32_t> tiles(B), blocks(B);
    std::vector<int64_t> rows(B);
    std::vector<double> share(B, 1.0);
    bool uneven_rows = false;
    for (int r = 0; r < B; ++r) {
      const ReqEntry &R = P.reqs[r];
      tiles[r] = R.tiles * (kTile / C.tile_keys);
      blocks[r] = d.n_kv_heads * ((R.lq * lp.group + rows_per_block - 1) / rows_per_block);
      rows[r] = (int64_t)R.lq * n_q_heads;
      uneven_rows |= blocks[r] != d.n_kv_heads * lp.nrb;
      // d128 row blocks end at the farthest limit of their rows: count the
      // part of the tiles they walk
      if (kern == Kern::Mfma128 && !P.doc_lim.empty() && R.ls == 0 && R.nlinks > 0) {
        const LinkEntry &last = P.links[R.link0 + R.nlinks - 1];
        share[r] = limit_share(P, R, lp.group, rows_per_block, last.tok0 + last.len);
      }
    }
    lp.skip_empty = kern == Kern::Mfma128 && !P.doc_lim.empty();
    const bool given = mode == Mode::Decode && num_splits > 0;
    if (given)
      C.req_splits.assign(B, num_splits);
    else
      C.req_splits = choose_splits(tiles, blocks, rows, share,
                                   split_cost(kern, s->shape.cus, d, P.max_rows, ss, uneven_rows));
    apply_splits(s, n_q_heads, rows_per_block, C);
    while (!given && C.part_bytes > kMostPartBytes && C.splits > 1) fewer_pieces(s, n_q_heads, C);
    // A decode call that the no-alloc entry takes (by its charge) fits its
    // scratch, also where uneven requests are cut into more pieces than the
    // charge counts or the work items need more than its slack. Cut here, for
    // both entries, so that their results are the same.
    if (mode == Mode::Decode && noalloc_charge(s, C, num_splits) <= kStaticScratchBytes)
      while (table_layout(C).bytes + C.work_bytes() > kStaticScratchBytes + kStaticScratchSlack &&
             C.splits > 1)
        fewer_pieces(s, n_q_heads, C);
    return PIC_OK;
  }

  int32_t splits = 1;
  const int64_t blocks = (int64_t)req->batch * d.n_kv_heads * lp.nrb;
  if (mode == Mode::Decode) {
    if (num_splits > 0) {
      splits = num_splits;
    } else {
      // eight workgroups per CU (stream kernel: one round), never more splits
      // than tiles
      const int64_t items = (kern == Kern::Stream ? ss.per_cu : 8) * (int64_t)s->shape.cus;
      splits = (int32_t)std::max<int64_t>(1, std::min<int64_t>((items + blocks - 1) / blocks, 256));
      splits = std::min(splits, std::max(1, P.max_tiles));
    }
  } else {
    // Vector-ALU and small calls, one split count for all requests: the
    // longest request's pieces no longer than the average work per resident
    // workgroup, at least min_piece tiles (1 for the vector-ALU kernel, whose
    // tiles are slow), at most 16 pieces.
    const int64_t slots = (int64_t)s->shape.cus * ss.per_cu;
    const int min_piece = kern == Kern::Stream ? 2 * ss.kpar : 1;
    int64_t work = 0;   // tiles summed over all non-empty workgroups
    for (const ReqEntry &R : P.reqs) {
      const int64_t rows = (int64_t)R.lq * lp.group;
      work += (int64_t)d.n_kv_heads * ((rows + rows_per_block - 1) / rows_per_block) * R.tiles;
    }
    const int64_t per_slot = std::max<int64_t>(min_piece, (work + slots - 1) / slots);
    splits = (int32_t)std::min<int64_t>(16, (P.max_tiles + per_slot - 1) / per_slot);
    // one workgroup per CU (lockstep, see choose_splits): as many pieces as
    // fill one round
    if (kern == Kern::Stream && ss.per_cu == 1 && blocks < slots)
      splits = std::max(splits, (int32_t)std::min<int64_t>(16, slots / blocks));
    splits = std::max(1, std::min(splits, P.max_tiles / min_piece));
  }
  C.splits = splits;
  lp.num_splits = splits;
  lp.spread = kern == Kern::Stream;
  C.part_rows = splits > 1 ? (int64_t)P.total_q * n_q_heads * splits : 0;
  C.part_off = round_up(P.own_bytes, 256);
  C.part_bytes = (size_t)C.part_rows * (d.d_v + 2) * sizeof(float);
  return PIC_OK;
}

// Enqueues a call whose tables are already on the device (lp.links, reqs,
// order set): own-KV staging, the attention kernel, the split combine.
// timed: the attention launch may be bracketed by the measurement events
// (pic_prof_begin); the entry point that allocates nothing passes false.
pic_status launch_call(const pic_store *s, const Setup &C, LinkParams lp, void *work,
                       const Prologue &pro, const void *q, const void *k_self,
                       const void *v_self, float scale, void *out, float *lse, hipStream_t st,
                       bool timed = true) {
  const pic_store_desc &d = s->desc;
  const bool mla = d.kind == PIC_MLA;
  lp.q = q;
  lp.k_self = k_self;
  lp.v_self = v_self;
  lp.out = out;
  lp.lse = lse;
  lp.scale_log2 = scale * 1.4426950408889634f;
  if (C.splits > 1) {
    lp.part_o = (float *)((char *)work + C.part_off);
    lp.part_m = lp.part_o + C.part_rows * d.d_v;
    lp.part_l = lp.part_m + C.part_rows;
  }
  if (C.P.max_own_lp > 0 || pro.copy_bytes > 0) {
    hipError_t e = launch_prologue(lp, pro.links, pro.reqs, mla, s->esz, C.P.max_own_lp,
                                   C.own_args.empty() ? nullptr : C.own_args.data(), work,
                                   pro.copy_src, pro.copy_dst, pro.copy_bytes, st);
    if (e != hipSuccess) return hip_fail(e, "prep_own_kernel");
  }
  std::pair<hipEvent_t, hipEvent_t> ev{nullptr, nullptr};
  const char *name = "";
  if (timed) prof_start(st, &ev);
  hipError_t e;
  if (C.kern == Kern::Decode128)
    e = launch_link_decode_d128(lp, st, &name);
  else if (C.kern == Kern::Mla)
    e = launch_link_mla(lp, st, &name);
  else if (C.kern == Kern::Mfma128)
    e = launch_link_mfma_d128(lp, st, &name);
  else if (C.kern == Kern::Stream)
    e = launch_link_stream(lp, d.dtype, C.stream_rows, st, &name);
  else
    e = launch_link_valu(lp, d.dtype, mla, st, &name);
  prof_stop(st, &ev, name);
  if (e != hipSuccess) return hip_fail(e, name);
  if (C.splits > 1) {
    e = launch_combine(lp, d.dtype, lp.max_rows * d.n_kv_heads, st);
    if (e != hipSuccess) return hip_fail(e, "combine_kernel");
  }
  return PIC_OK;
}

// A small call's kernels: the tables go as a kernel argument and the own KV
// is read in place, so the only device memory besides the caller's tensors
// is `work` for the split partials (C.part_bytes, unused when not split).
// links: host, C.P.links.size() entries (C.P.links, or a plan's for one
// layer).
pic_status launch_small(const pic_store_desc &d, const Setup &C, const LinkEntry *links,
                        void *work, const void *q, const void *k_self, const void *v_self,
                        float scale, void *out, float *lse, hipStream_t st) {
  LinkParams lp = C.lp;
  if (C.splits > 1) {
    lp.part_o = (float *)work;
    lp.part_m = lp.part_o + C.part_rows * d.d_v;
    lp.part_l = lp.part_m + C.part_rows;
  }
  lp.links = nullptr;
  lp.items = nullptr;
  lp.reqs = nullptr;
  lp.order = nullptr;
  lp.comb = nullptr;
  lp.doc_lim = nullptr;
  lp.q = q;
  lp.k_self = k_self;
  lp.v_self = v_self;
  lp.out = out;
  lp.lse = lse;
  lp.scale_log2 = scale * 1.4426950408889634f;
  std::pair<hipEvent_t, hipEvent_t> ev{nullptr, nullptr};
  const char *name = "";
  hipError_t e;
  if (C.lean) {
    LeanTabs t;
    memset(&t, 0, sizeof(t));
    std::copy(links, links + C.P.links.size(), t.links);
    int32_t base = 0;
    for (size_t i = 0; i < C.P.order.size(); ++i) {
      const ReqEntry &R = C.P.reqs[C.P.order[i]];
      t.reqs[i] = R;
      t.tile_base[i] = base;
      for (int32_t k = 0; k < R.nlinks; ++k) {
        const LinkEntry &L = links[R.link0 + k];
        const int32_t n = (L.len + kTile - 1) / kTile;
        for (int32_t j = 0; j < n; ++j) t.tile_link[base + L.tile0 + j] = (uint8_t)k;
      }
      base += R.tiles;
    }
    prof_start(st, &ev);
    e = launch_link_lean(lp, t, d.dtype, st, &name);
  } else {
    SmallTabs t;
    memset(&t, 0, sizeof(t));
    std::copy(links, links + C.P.links.size(), t.links);
    std::copy(C.P.reqs.begin(), C.P.reqs.end(), t.reqs);
    std::copy(C.P.order.begin(), C.P.order.end(), t.order);
    prof_start(st, &ev);
    e = C.kern == Kern::Stream
            ? launch_link_stream_small(lp, t, d.dtype, C.stream_rows, st, &name)
            : launch_link_small(lp, t, d.dtype, d.kind == PIC_MLA, st, &name);
  }
  prof_stop(st, &ev, name);
  if (e != hipSuccess) return hip_fail(e, name);
  if (C.splits > 1) {
    e = launch_combine(lp, d.dtype, lp.max_rows * d.n_kv_heads, st);
    if (e != hipSuccess) return hip_fail(e, "combine_kernel");
  }
  return PIC_OK;
}

pic_status small_link_call(pic_store *s, const Setup &C, const void *q, const void *k_self,
                           const void *v_self, float scale, void *out, float *lse,
                           hipStream_t st) {
  Stage *stage = nullptr;
  pic_status rc = stage_acquire(s, 0, &stage);
  if (rc != PIC_OK) return rc;
  if (C.splits > 1) {
    rc = ensure_work(stage, C.part_bytes);
    if (rc != PIC_OK) return rc;
  }
  rc = launch_small(s->desc, C, C.P.links.data(), stage->work, q, k_self, v_self, scale, out,
                    lse, st);
  if (rc != PIC_OK) return rc;
  HIP_TRY(hipEventRecord(stage->done, st), "hipEventRecord(stage)");
  stage->pending = true;
  return PIC_OK;
}

pic_status link_call(pic_store *s, const pic_link_req *req, int32_t n_q_heads, const void *q,
                     const void *k_self, const void *v_self, float scale, int32_t num_splits,
                     void *out, float *lse, void *stream, Mode mode) {
  if (!req) return fail(PIC_ERR_INVALID, "req is NULL");
  Setup C;
  pic_status rc = setup_call(s, req, n_q_heads, scale, req->layer, num_splits, mode, C);
  if (rc != PIC_OK) return rc;
  if (req->batch == 0) return PIC_OK;
  rc = check_tensors(s, C.P, q, k_self, v_self, out);
  if (rc != PIC_OK) return rc;
  if (C.P.total_q == 0) return PIC_OK;
  const hipStream_t st = (hipStream_t)stream;
  // the workspace is allocated on the store's device
  DeviceGuard dg(s->device);
  if (!dg.ok) return fail(PIC_ERR_HIP, "cannot select the store's device");
  if (C.small) return small_link_call(s, C, q, k_self, v_self, scale, out, lse, st);
  Stage *stage = nullptr;
  TableLayout tl;
  LinkParams lp = C.lp;
  rc = upload(s, C, &stage, lp, tl);
  if (rc != PIC_OK) return rc;
  Prologue pro;
  const char *hd = (const char *)stage->host_dev;
  pro.links = (const LinkEntry *)hd;
  pro.reqs = (const ReqEntry *)(hd + tl.off_r);
  pro.copy_src = hd;
  pro.copy_dst = stage->dev;
  pro.copy_bytes = (int64_t)tl.bytes;
  rc = launch_call(s, C, lp, stage->work, pro, q, k_self, v_self, scale, out, lse, st);
  if (rc != PIC_OK) return rc;
  HIP_TRY(hipEventRecord(stage->done, st), "hipEventRecord(stage)");
  stage->pending = true;
  return PIC_OK;
}

}  // namespace

// A request batch resolved once for repeated calls: the link tables of every
// layer and the call's workspace live on the device for the plan's lifetime.
struct pic_link_plan {
  pic_store *store = nullptr;
  Setup C;
  int32_t batch = 0;
  void *dev = nullptr;           // [layer tables][workspace]
  size_t table_bytes = 0;        // one layer's tables, 256-byte aligned
  TableLayout layout{};          // within a layer's tables
  void *work = nullptr;          // inside dev
  // small calls (see small_tables): every layer's link table on the host,
  // [layer][link], run by the small-call kernels as pic_link_attn /
  // pic_link_decode run them (tables as a kernel argument)
  bool small = false;
  std::vector<LinkEntry> small_links;
};

extern "C" {

pic_status pic_store_create(const pic_store_desc *desc, pic_store **out) {
  if (!desc || !out) return fail(PIC_ERR_INVALID, "desc/out is NULL");
  *out = nullptr;
  const pic_store_desc &d = *desc;
  if (d.kind != PIC_GQA && d.kind != PIC_MLA) return fail(PIC_ERR_INVALID, "unknown kind %d", d.kind);
  if (d.dtype != PIC_F32 && d.dtype != PIC_BF16) return fail(PIC_ERR_INVALID, "unknown dtype %d", d.dtype);
  if (d.n_layers < 0 || d.n_layers > 256) return fail(PIC_ERR_INVALID, "n_layers must be 0..256");
  if (d.n_kv_heads <= 0 || d.d_k <= 0 || d.d_v <= 0 || d.capacity_tokens <= 0)
    return fail(PIC_ERR_INVALID, "n_kv_heads, d_k, d_v and capacity_tokens must be positive");
  if (d.kind == PIC_MLA && (d.n_kv_heads != 1 || d.d_v > d.d_k))
    return fail(PIC_ERR_INVALID, "MLA needs n_kv_heads == 1 and d_v <= d_k");
  if (d.d_k % 8 || d.d_v % 8) return fail(PIC_ERR_UNSUPPORTED, "d_k and d_v must be multiples of 8");
  if (d.d_k > 1024 || d.d_v > 1024 || d.n_kv_heads > 256)
    return fail(PIC_ERR_UNSUPPORTED, "head count or width too large");
  pic_store *s = new (std::nothrow) pic_store();
  if (!s) return fail(PIC_ERR_OOM, "host allocation failed");
  s->desc = d;
  s->esz = d.dtype == PIC_F32 ? 4 : 2;
  s->capacity = round_up(d.capacity_tokens, kTile);
  s->k_tok_elems = (int64_t)d.n_kv_heads * d.d_k;
  s->v_tok_elems = d.kind == PIC_GQA ? (int64_t)d.n_kv_heads * d.d_v : 0;
  s->n_layers = d.n_layers > 1 ? d.n_layers : 1;
  s->layer_bytes = s->capacity * (s->k_tok_elems + s->v_tok_elems) * s->esz;
  s->free_runs.emplace(0, s->capacity / kTile);
  hipError_t e = hipGetDevice(&s->device);
  if (e == hipSuccess) s->shape = device_shape();
  if (e == hipSuccess) e = hipMalloc((void **)&s->pool, (size_t)s->layer_bytes * s->n_layers);
  if (e != hipSuccess) {
    delete s;
    return hip_fail(e, "hipMalloc(pool)");
  }
  try {
    s->page_refs.assign((size_t)(s->capacity / kTile), 0);
  } catch (...) {
    (void)hipFree(s->pool);
    delete s;
    return fail(PIC_ERR_OOM, "host allocation failed");
  }
  *out = s;
  return PIC_OK;
}

pic_status pic_store_destroy(pic_store *s) {
  if (!s) return PIC_OK;
  if (s->live_plans > 0)
    return fail(PIC_ERR_INVALID, "%lld link plans of this store are still alive",
                (long long)s->live_plans);
  DeviceGuard dg(s->device);
  (void)hipDeviceSynchronize();
  for (Stage &st : s->ring) {
    if (st.host) (void)hipHostFree(st.host);
    if (st.dev) (void)hipFree(st.dev);
    if (st.work) (void)hipFree(st.work);
    if (st.done) (void)hipEventDestroy(st.done);
  }
  for (auto &pr : s->pending) (void)hipEventDestroy(pr.first);
  if (s->pool) {
    if (s->imported)
      (void)hipIpcCloseMemHandle(s->pool);
    else
      (void)hipFree(s->pool);
  }
  delete s;
  return PIC_OK;
}

pic_status pic_store_put(pic_store *s, uint64_t chunk_id, int64_t n_tokens, const void *k,
                         const void *v, void *stream) {
  if (!s) return fail(PIC_ERR_INVALID, "store is NULL");
  if (s->imported) return fail(PIC_ERR_INVALID, "the store was imported from another process and is read-only");
  if (n_tokens <= 0 || n_tokens > INT32_MAX / 4) return fail(PIC_ERR_INVALID, "n_tokens out of range");
  if (!k) return fail(PIC_ERR_INVALID, "k is NULL");
  const bool gqa = s->desc.kind == PIC_GQA;
  if (gqa && !v) return fail(PIC_ERR_INVALID, "v is NULL");
  if (!gqa && v) return fail(PIC_ERR_INVALID, "v must be NULL for MLA");
  if (s->map.count(chunk_id)) return fail(PIC_ERR_EXISTS, "chunk id 0x%llx already stored",
                                          (unsigned long long)chunk_id);
  const int64_t pages = round_up(n_tokens, kTile) / kTile;
  DeviceGuard dg(s->device);
  if (!dg.ok) return fail(PIC_ERR_HIP, "cannot select the store's device");
  for (const void *ptr : {k, v}) {
    if (!ptr) continue;
    hipPointerAttribute_t attr;
    if (hipPointerGetAttributes(&attr, ptr) != hipSuccess ||
        (attr.type != hipMemoryTypeDevice && attr.type != hipMemoryTypeManaged)) {
      (void)hipGetLastError();
      return fail(PIC_ERR_INVALID, "k and v must be device memory");
    }
  }
  std::vector<Run> runs;
  pic_status rc = take_pages(s, pages, runs);
  if (rc != PIC_OK) return rc;
  int32_t tok = 0;
  for (Run &r : runs) {
    r.tok0 = tok;
    r.ntok = (int32_t)std::min<int64_t>((int64_t)r.pages * kTile, n_tokens - tok);
    tok += r.ntok;
  }
  const hipStream_t st = (hipStream_t)stream;
  const pic_store_desc &d = s->desc;
  // layer l of the caller's buffers -> layer l of each run
  const int64_t k_src_layer = n_tokens * s->k_tok_elems * s->esz;
  const int64_t v_src_layer = n_tokens * s->v_tok_elems * s->esz;
  hipError_t e = hipSuccess;
  for (const Run &r : runs) {
    const LinkEntry E = run_entry(s, r, 0);
    PutParams pp{};
    pp.src_k = (const char *)k + (int64_t)r.tok0 * s->k_tok_elems * s->esz;
    pp.src_v = gqa ? (const char *)v + (int64_t)r.tok0 * s->v_tok_elems * s->esz : nullptr;
    pp.dst_k = (char *)E.k;
    pp.dst_v = (char *)E.v;
    pp.src_k_layer = k_src_layer;
    pp.src_v_layer = v_src_layer;
    pp.layer_bytes = s->layer_bytes;
    pp.n_tokens = r.ntok;
    pp.lp = E.lp;
    pp.heads = d.n_kv_heads;
    pp.d_k = d.d_k;
    pp.d_v = d.d_v;
    pp.esz = s->esz;
    e = launch_put(pp, s->n_layers, st);
    if (e != hipSuccess) break;
  }
  if (e != hipSuccess) {
    for (const Run &r : runs) free_run(s, r.page0, r.pages);
    return hip_fail(e, "put kernels");
  }
  Slot sl;
  sl.len = n_tokens;
  for (const Run &r : runs) s->block_refs[r.page0] = 1;
  ref_pages(s, runs, 1);
  sl.runs = std::move(runs);
  s->used += pages * kTile;
  s->map.emplace(chunk_id, std::move(sl));
  return PIC_OK;
}

pic_status pic_store_derive(pic_store *s, uint64_t new_id, uint64_t base_id, int32_t n_rows,
                            const int32_t *rows, void *stream) {
  if (!s) return fail(PIC_ERR_INVALID, "store is NULL");
  if (s->imported) return fail(PIC_ERR_INVALID, "the store was imported from another process and is read-only");
  auto bit = s->map.find(base_id);
  if (bit == s->map.end()) return fail(PIC_ERR_NOT_FOUND, "base chunk id 0x%llx not in the store",
                                       (unsigned long long)base_id);
  if (s->map.count(new_id)) return fail(PIC_ERR_EXISTS, "chunk id 0x%llx already stored",
                                        (unsigned long long)new_id);
  const int64_t len = bit->second.len;
  if (!check_rows(rows, n_rows, len))
    return fail(PIC_ERR_INVALID, "rows must be strictly increasing and below the chunk's %lld tokens",
                (long long)len);
  const int64_t npages = round_up(len, kTile) / kTile;
  std::vector<char> own(npages, 0);
  int64_t n_own = 0;
  for (int32_t i = 0; i < n_rows; ++i) {
    char &o = own[rows[i] / kTile];
    n_own += !o;
    o = 1;
  }
  DeviceGuard dg(s->device);
  if (!dg.ok) return fail(PIC_ERR_HIP, "cannot select the store's device");
  std::vector<Run> fresh;
  pic_status rc = take_pages(s, n_own, fresh);
  if (rc != PIC_OK) return rc;
  const Slot &B = s->map.at(base_id);   // take_pages does not touch the map
  // One view per chunk page, merged where consecutive pages are consecutive
  // pages of one block; private pages take the fresh blocks' pages in order.
  std::vector<Run> views;
  std::vector<std::pair<Run, Run>> copies;     // (source page view, destination page view)
  size_t fb = 0;
  int32_t fq = 0;
  for (int64_t p = 0; p < npages; ++p) {
    const int32_t t0 = (int32_t)(p * kTile);
    const int32_t nt = (int32_t)std::min<int64_t>(kTile, len - t0);
    const Run &src = view_of(B, t0);
    Run pv{src.page0, src.pages, t0, nt, src.skip + (t0 - src.tok0) / kTile};
    if (own[p]) {
      Run dst{fresh[fb].page0, fresh[fb].pages, t0, nt, fq};
      copies.emplace_back(pv, dst);
      pv = dst;
      if (++fq == fresh[fb].pages) {
        ++fb;
        fq = 0;
      }
    }
    if (!views.empty()) {
      Run &last = views.back();
      if (last.page0 == pv.page0 && last.skip + last.ntok / kTile == pv.skip && last.ntok % kTile == 0) {
        last.ntok += nt;
        continue;
      }
    }
    views.push_back(pv);
  }
  // copy the private pages' base content, every layer (K rows of each head,
  // V^T columns of each head and dim)
  const hipStream_t st = (hipStream_t)stream;
  const pic_store_desc &d = s->desc;
  hipError_t e = hipSuccess;
  for (size_t c0 = 0; c0 < copies.size() && e == hipSuccess; c0 += kCopyPages) {
    const size_t n = std::min<size_t>(kCopyPages, copies.size() - c0);
    PageCopies pc;
    pc.layer_bytes = s->layer_bytes;
    pc.heads = d.n_kv_heads;
    pc.d_k = d.d_k;
    pc.d_v = d.d_v;
    pc.esz = s->esz;
    for (size_t i = 0; i < n; ++i) {
      const LinkEntry S = run_entry(s, copies[c0 + i].first, 0), D = run_entry(s, copies[c0 + i].second, 0);
      const bool gqa = d.kind == PIC_GQA;
      pc.page[i] = PageCopy{(const char *)S.k, gqa ? (const char *)S.v : nullptr, (char *)D.k,
                            gqa ? (char *)D.v : nullptr, S.lp, D.lp};
    }
    e = launch_copy_pages(pc, (int32_t)n, s->n_layers, st);
  }
  if (e != hipSuccess) {
    for (const Run &r : fresh) free_run(s, r.page0, r.pages);
    return hip_fail(e, "derive page copies");
  }
  for (const Run &r : fresh) s->block_refs[r.page0] = 0;
  std::vector<int64_t> blocks;
  for (const Run &v : views) blocks.push_back(v.page0);
  std::sort(blocks.begin(), blocks.end());
  blocks.erase(std::unique(blocks.begin(), blocks.end()), blocks.end());
  for (int64_t b : blocks) ++s->block_refs.at(b);
  ref_pages(s, views, 1);
  s->used += n_own * kTile;
  Slot sl;
  sl.len = len;
  sl.runs = std::move(views);
  sl.derived = true;
  s->map.emplace(new_id, std::move(sl));
  return PIC_OK;
}

pic_status pic_store_write_rows(pic_store *s, uint64_t chunk_id, int32_t layer, int32_t n_rows,
                                const int32_t *rows, const void *k, const void *v, void *stream) {
  if (!s) return fail(PIC_ERR_INVALID, "store is NULL");
  if (s->imported) return fail(PIC_ERR_INVALID, "the store was imported from another process and is read-only");
  auto it = s->map.find(chunk_id);
  if (it == s->map.end()) return fail(PIC_ERR_NOT_FOUND, "chunk id 0x%llx not in the store",
                                      (unsigned long long)chunk_id);
  const Slot &sl = it->second;
  if (!sl.derived)
    return fail(PIC_ERR_INVALID, "chunk id 0x%llx was not made by pic_store_derive",
                (unsigned long long)chunk_id);
  if (layer < 0 || layer >= s->n_layers)
    return fail(PIC_ERR_INVALID, "layer %d outside the store's %d layers", layer, s->n_layers);
  if (!check_rows(rows, n_rows, sl.len))
    return fail(PIC_ERR_INVALID, "rows must be strictly increasing and below the chunk's %lld tokens",
                (long long)sl.len);
  if (n_rows == 0) return PIC_OK;
  const bool gqa = s->desc.kind == PIC_GQA;
  if (!k || (gqa && !v)) return fail(PIC_ERR_INVALID, "k/v is NULL");
  if (!gqa && v) return fail(PIC_ERR_INVALID, "v must be NULL for MLA");
  for (int32_t i = 0; i < n_rows; ++i) {
    const Run &r = view_of(sl, rows[i]);
    if (s->page_refs[r.page0 + r.skip + (rows[i] - r.tok0) / kTile] != 1)
      return fail(PIC_ERR_INVALID, "row %d of chunk 0x%llx is on a page shared with another chunk",
                  rows[i], (unsigned long long)chunk_id);
  }
  DeviceGuard dg(s->device);
  if (!dg.ok) return fail(PIC_ERR_HIP, "cannot select the store's device");
  const pic_store_desc &d = s->desc;
  // one launch per kWriteRowsMost rows or kWriteViews of the views they lie in
  RowView views[kWriteViews];
  size_t v0 = 0;                     // the view after the last one listed
  int32_t n_views = 0, first = 0;    // views listed, first row not yet written
  auto flush = [&](int32_t end) {
    const int64_t done = first;
    const hipError_t e = launch_write_rows(
        views, n_views, rows + first, end - first,
        (const char *)k + done * s->k_tok_elems * s->esz,
        gqa ? (const char *)v + done * s->v_tok_elems * s->esz : nullptr, d.n_kv_heads, d.d_k,
        d.d_v, s->esz, (hipStream_t)stream);
    first = end;
    n_views = 0;
    return e;
  };
  for (int32_t i = 0; i < n_rows; ++i) {
    const bool listed = n_views > 0 && rows[i] < sl.runs[v0 - 1].tok0 + sl.runs[v0 - 1].ntok;
    if (i - first == kWriteRowsMost || (!listed && n_views == kWriteViews))
      HIP_TRY(flush(i), "write_rows_kernel");
    if (listed && n_views > 0) continue;
    v0 = 0;
    while (rows[i] >= sl.runs[v0].tok0 + sl.runs[v0].ntok) ++v0;
    const LinkEntry E = run_entry(s, sl.runs[v0], layer);
    views[n_views++] = RowView{(void *)E.k, gqa ? (void *)E.v : nullptr, E.lp, sl.runs[v0].tok0};
    ++v0;
  }
  HIP_TRY(flush(n_rows), "write_rows_kernel");
  return PIC_OK;
}

pic_status pic_store_remove(pic_store *s, uint64_t chunk_id, void *stream) {
  if (!s) return fail(PIC_ERR_INVALID, "store is NULL");
  if (s->imported) return fail(PIC_ERR_INVALID, "the store was imported from another process and is read-only");
  auto it = s->map.find(chunk_id);
  if (it == s->map.end()) return fail(PIC_ERR_NOT_FOUND, "chunk id 0x%llx not in the store",
                                      (unsigned long long)chunk_id);
  if (it->second.plan_refs > 0)
    return fail(PIC_ERR_INVALID, "chunk id 0x%llx is linked by %lld live link plans",
                (unsigned long long)chunk_id, (long long)it->second.plan_refs);
  DeviceGuard dg(s->device);
  if (!dg.ok) return fail(PIC_ERR_HIP, "cannot select the store's device");
  // the pages are reused only after the work enqueued so far on `stream`
  // (the calls that may read them) has completed
  hipEvent_t ev = nullptr;
  HIP_TRY(hipEventCreateWithFlags(&ev, hipEventDisableTiming), "hipEventCreate(remove)");
  hipError_t e = hipEventRecord(ev, (hipStream_t)stream);
  if (e != hipSuccess) {
    (void)hipEventDestroy(ev);
    return hip_fail(e, "hipEventRecord(remove)");
  }
  // blocks no other chunk views are freed once the event has completed
  ref_pages(s, it->second.runs, -1);
  std::vector<Run> freed;
  std::vector<int64_t> blocks;
  for (const Run &r : it->second.runs) blocks.push_back(r.page0);
  std::sort(blocks.begin(), blocks.end());
  blocks.erase(std::unique(blocks.begin(), blocks.end()), blocks.end());
  for (int64_t b : blocks) {
    auto ref = s->block_refs.find(b);
    if (--ref->second > 0) continue;
    const Run &r = *std::find_if(it->second.runs.begin(), it->second.runs.end(),
                                 [b](const Run &x) { return x.page0 == b; });
    freed.push_back(Run{r.page0, r.pages, 0, 0});
    s->block_refs.erase(ref);
  }
  if (freed.empty())
    (void)hipEventDestroy(ev);
  else
    s->pending.emplace_back(ev, std::move(freed));
  s->map.erase(it);
  return PIC_OK;
}

namespace {

// Layout of an exported store: header, then per chunk its record and runs.
constexpr uint64_t kExportMagic = 0x31524f5453434950ull;   // "PICSTOR1"
struct ExportHeader {
  uint64_t magic;
  uint64_t bytes;                // whole blob
  pic_store_desc desc;
  int64_t capacity, layer_bytes, k_tok_elems, v_tok_elems, used, n_chunks;
  int32_t n_layers, esz;
  hipIpcMemHandle_t handle;      // the pool
};
struct ExportChunk {
  uint64_t id;
  int64_t len;
  int32_t n_runs, derived;
};
struct ExportRun {
  int64_t page0;
  int32_t pages, tok0, ntok, skip;
};

// Pools from 2 GiB up are not exported: opening such a mapping in another
// process has not returned on the target machines.
constexpr int64_t kMaxExportBytes = (int64_t(1) << 31) - 1;

size_t export_size(const pic_store *s) {
  size_t n = sizeof(ExportHeader);
  for (const auto &kv : s->map) n += sizeof(ExportChunk) + kv.second.runs.size() * sizeof(ExportRun);
  return n;
}

}  // namespace

pic_status pic_store_export(pic_store *s, void *buf, size_t buf_bytes, size_t *bytes_out) {
  if (!s || !bytes_out) return fail(PIC_ERR_INVALID, "store/bytes_out is NULL");
  if (s->imported) return fail(PIC_ERR_INVALID, "an imported store cannot be exported again");
  const int64_t pool_bytes = s->layer_bytes * s->n_layers;
  if (pool_bytes > kMaxExportBytes)
    return fail(PIC_ERR_UNSUPPORTED, "pool of %lld bytes: only pools below 2 GiB are exported",
                (long long)pool_bytes);
  const size_t need = export_size(s);
  *bytes_out = need;
  if (!buf) return PIC_OK;
  if (buf_bytes < need) return fail(PIC_ERR_INVALID, "buffer of %zu bytes, %zu needed", buf_bytes, need);
  DeviceGuard dg(s->device);
  if (!dg.ok) return fail(PIC_ERR_HIP, "cannot select the store's device");
  // every put and copy enqueued so far lands before another process reads
  HIP_TRY(hipDeviceSynchronize(), "hipDeviceSynchronize(export)");
  ExportHeader h{};
  h.magic = kExportMagic;
  h.bytes = need;
  h.desc = s->desc;
  h.capacity = s->capacity;
  h.layer_bytes = s->layer_bytes;
  h.k_tok_elems = s->k_tok_elems;
  h.v_tok_elems = s->v_tok_elems;
  h.used = s->used;
  h.n_chunks = (int64_t)s->map.size();
  h.n_layers = s->n_layers;
  h.esz = s->esz;
  HIP_TRY(hipIpcGetMemHandle(&h.handle, s->pool), "hipIpcGetMemHandle(pool)");
  char *o = (char *)buf;
  memcpy(o, &h, sizeof h);
  o += sizeof h;
  for (const auto &kv : s->map) {
    const ExportChunk ch{kv.first, kv.second.len, (int32_t)kv.second.runs.size(),
                         kv.second.derived ? 1 : 0};
    memcpy(o, &ch, sizeof ch);
    o += sizeof ch;
    for (const Run &r : kv.second.runs) {
      const ExportRun er{r.page0, r.pages, r.tok0, r.ntok, r.skip};
      memcpy(o, &er, sizeof er);
      o += sizeof er;
    }
  }
  return PIC_OK;
}

pic_status pic_store_import(const void *buf, size_t buf_bytes, pic_store **out) {
  if (!buf || !out) return fail(PIC_ERR_INVALID, "buf/out is NULL");
  *out = nullptr;
  ExportHeader h;
  if (buf_bytes < sizeof h) return fail(PIC_ERR_INVALID, "blob too short");
  memcpy(&h, buf, sizeof h);
  if (h.magic != kExportMagic) return fail(PIC_ERR_INVALID, "not an exported store");
  if (h.bytes > buf_bytes || h.n_chunks < 0 || h.n_layers < 1 || h.n_layers > 256 ||
      (h.esz != 2 && h.esz != 4) || h.capacity <= 0 || h.capacity % kTile ||
      h.layer_bytes != h.capacity * (h.k_tok_elems + h.v_tok_elems) * h.esz ||
      h.layer_bytes * h.n_layers > kMaxExportBytes)
    return fail(PIC_ERR_INVALID, "inconsistent exported store header");
  const int64_t pages = h.capacity / kTile;
  pic_store *s = new (std::nothrow) pic_store();
  if (!s) return fail(PIC_ERR_OOM, "host allocation failed");
  s->desc = h.desc;
  s->esz = h.esz;
  s->capacity = h.capacity;
  s->used = h.used;
  s->k_tok_elems = h.k_tok_elems;
  s->v_tok_elems = h.v_tok_elems;
  s->n_layers = h.n_layers;
  s->layer_bytes = h.layer_bytes;
  const char *in = (const char *)buf + sizeof h, *end = (const char *)buf + h.bytes;
  for (int64_t c = 0; c < h.n_chunks; ++c) {
    ExportChunk ch;
    if (in + sizeof ch > end) break;
    memcpy(&ch, in, sizeof ch);
    in += sizeof ch;
    if (ch.n_runs < 1 || ch.len < 1 || in + (size_t)ch.n_runs * sizeof(ExportRun) > end) {
      delete s;
      return fail(PIC_ERR_INVALID, "corrupt chunk record in the exported store");
    }
    Slot sl;
    sl.len = ch.len;
    sl.derived = ch.derived != 0;
    int64_t covered = 0;
    for (int32_t i = 0; i < ch.n_runs; ++i) {
      ExportRun er;
      memcpy(&er, in, sizeof er);
      in += sizeof er;
      // every view lies inside the pool and the views cover the chunk in order
      if (er.page0 < 0 || er.pages < 1 || er.page0 + er.pages > pages || er.skip < 0 ||
          er.ntok < 1 || er.tok0 != covered ||
          (int64_t)er.skip * kTile + er.ntok > (int64_t)er.pages * kTile) {
        delete s;
        return fail(PIC_ERR_INVALID, "corrupt run in the exported store");
      }
      covered += er.ntok;
      sl.runs.push_back(Run{er.page0, er.pages, er.tok0, er.ntok, er.skip});
    }
    if (covered != ch.len || !s->map.emplace(ch.id, std::move(sl)).second) {
      delete s;
      return fail(PIC_ERR_INVALID, "corrupt chunk record in the exported store");
    }
  }
  if ((int64_t)s->map.size() != h.n_chunks) {
    delete s;
    return fail(PIC_ERR_INVALID, "truncated exported store");
  }
  hipError_t e = hipGetDevice(&s->device);
  if (e == hipSuccess) {
    s->shape = device_shape();
    e = hipIpcOpenMemHandle((void **)&s->pool, h.handle, hipIpcMemLazyEnablePeerAccess);
  }
  if (e != hipSuccess) {
    delete s;
    return hip_fail(e, "hipIpcOpenMemHandle(pool)");
  }
  s->imported = true;
  *out = s;
  return PIC_OK;
}

pic_status pic_store_lookup(const pic_store *s, uint64_t chunk_id, int64_t *n_tokens_out) {
  if (!s || !n_tokens_out) return fail(PIC_ERR_INVALID, "store/n_tokens_out is NULL");
  auto it = s->map.find(chunk_id);
  if (it == s->map.end()) return fail(PIC_ERR_NOT_FOUND, "chunk id 0x%llx not in the store",
                                      (unsigned long long)chunk_id);
  *n_tokens_out = it->second.len;
  return PIC_OK;
}

pic_status pic_store_usage(const pic_store *s, int64_t *used, int64_t *cap, int64_t *n) {
  if (!s) return fail(PIC_ERR_INVALID, "store is NULL");
  if (used) *used = s->used;
  if (cap) *cap = s->capacity;
  if (n) *n = (int64_t)s->map.size();
  return PIC_OK;
}

pic_status pic_link_attn(pic_store *s, const pic_link_req *req, int32_t n_q_heads, const void *q,
                         const void *k_self, const void *v_self, float softmax_scale, void *out,
                         float *lse, void *stream) {
  return link_call(s, req, n_q_heads, q, k_self, v_self, softmax_scale, 0, out, lse, stream,
                   Mode::Prefill);
}

pic_status pic_link_decode(pic_store *s, const pic_link_req *req, int32_t n_q_heads,
                           const void *q, const void *k_self, const void *v_self,
                           float softmax_scale, int32_t num_splits, void *out, float *lse,
                           void *stream) {
  return link_call(s, req, n_q_heads, q, k_self, v_self, softmax_scale, num_splits, out, lse,
                   stream, Mode::Decode);
}

pic_status pic_link_decode_noalloc(pic_store *s, const pic_link_req *req, int32_t n_q_heads,
                                   const void *q, const void *k_self, const void *v_self,
                                   float softmax_scale, int32_t num_splits, void *out, float *lse,
                                   void *stream) {
  if (!req) return fail(PIC_ERR_INVALID, "req is NULL");
  Setup C;
  pic_status rc = setup_call(s, req, n_q_heads, softmax_scale, req->layer, num_splits,
                             Mode::Decode, C);
  if (rc != PIC_OK) return rc;
  if (req->batch == 0) return PIC_OK;
  rc = check_tensors(s, C.P, q, k_self, v_self, out);
  if (rc != PIC_OK) return rc;
  if (C.P.total_q == 0) return PIC_OK;
  // (A small call runs the kernels pic_link_decode runs for it, tables as a
  // kernel argument and own KV read in place: the scratch holds only its
  // split partials.)
  const size_t charge = noalloc_charge(s, C, num_splits);
  if (charge > kStaticScratchBytes)
    return fail(PIC_ERR_INVALID,
                "the call needs %zu bytes of scratch (tables, own KV, split partials); the static "
                "scratch holds %zu", charge, kStaticScratchBytes);
  if (C.small) {
    // What a given split count needs is what it is charged for; the stream
    // kernel's own choice stays below it (fewer than 1024 workgroups of at
    // most 128 rows x 66 or 64 x 130 floats: 35 MB).
    if (C.part_bytes > kStaticScratchBytes)
      return fail(PIC_ERR_INVALID, "the call's split partials exceed the static scratch");
    DeviceGuard dg(s->device);
    if (!dg.ok) return fail(PIC_ERR_HIP, "cannot select the store's device");
    void *base = nullptr;
    HIP_TRY(static_scratch(&base), "hipGetSymbolAddress(scratch)");
    return launch_small(s->desc, C, C.P.links.data(), base, q, k_self, v_self, softmax_scale,
                        out, lse, (hipStream_t)stream);
  }
  // scratch layout: [tables][workspace] (setup_call cut the pieces to fit)
  const TableLayout t = table_layout(C);
  if (t.bytes + C.work_bytes() > kStaticScratchBytes + kStaticScratchSlack)
    return fail(PIC_ERR_INVALID, "the call's tables exceed the static scratch");
  DeviceGuard dg(s->device);
  if (!dg.ok) return fail(PIC_ERR_HIP, "cannot select the store's device");
  void *base = nullptr;
  HIP_TRY(static_scratch(&base), "hipGetSymbolAddress(scratch)");
  char *dev = (char *)base;
  place_own(s, C.P, dev + t.bytes, C.P.links.data());
  std::vector<char> host(t.bytes, 0);
  write_tables(C, t, C.P.links.data(), host.data());
  const hipStream_t st = (hipStream_t)stream;
  // pageable source: the runtime copies it before returning (no staging
  // buffer of ours, no allocation)
  HIP_TRY(hipMemcpyAsync(dev, host.data(), t.bytes, hipMemcpyHostToDevice, st),
          "hipMemcpyAsync(tables to scratch)");
  LinkParams lp = C.lp;
  point_tables(C, t, dev, lp);
  Prologue pro;
  pro.links = lp.links;
  pro.reqs = lp.reqs;
  return launch_call(s, C, lp, dev + t.bytes, pro, q, k_self, v_self, softmax_scale, out, lse, st,
                     false);
}

pic_status pic_link_plan_create(pic_store *s, const pic_link_req *req, int32_t n_q_heads,
                                int32_t mode, int32_t num_splits, pic_link_plan **out) {
  if (!out) return fail(PIC_ERR_INVALID, "out is NULL");
  *out = nullptr;
  if (!s) return fail(PIC_ERR_INVALID, "store is NULL");
  if (!req) return fail(PIC_ERR_INVALID, "req is NULL");
  if (req->layer != 0) return fail(PIC_ERR_INVALID, "req->layer must be 0 (each run names its layer)");
  if (mode != PIC_PREFILL && mode != PIC_DECODE) return fail(PIC_ERR_INVALID, "unknown mode %d", mode);
  if (mode == PIC_PREFILL && num_splits != 0)
    return fail(PIC_ERR_INVALID, "num_splits must be 0 for prefill plans");
  pic_link_plan *pl = new (std::nothrow) pic_link_plan();
  if (!pl) return fail(PIC_ERR_OOM, "host allocation failed");
  // the scale only has to pass validation here; each run passes its own
  pic_status rc = setup_call(s, req, n_q_heads, 1.0f, 0, num_splits,
                             mode == PIC_DECODE ? Mode::Decode : Mode::Prefill, pl->C);
  if (rc != PIC_OK) {
    delete pl;
    return rc;
  }
  pl->store = s;
  pl->batch = req->batch;
  const Plan &P = pl->C.P;
  const size_t nl = P.links.size();
  pl->layout = table_layout(pl->C);
  pl->table_bytes = pl->layout.bytes;
  // A small call keeps its tables on the host (one per layer) and needs
  // device memory for its split partials only.
  pl->small = pl->C.small;
  if (pl->small) {
    pl->small_links.resize((size_t)s->n_layers * nl);
    std::vector<bool> own_link(nl, false);
    for (auto &o : P.own) own_link[o.first] = true;
    for (int32_t l = 0; l < s->n_layers; ++l)
      for (size_t i = 0; i < nl; ++i) {
        LinkEntry E = P.links[i];
        if (!own_link[i]) {
          E.k = (const char *)E.k + (int64_t)l * s->layer_bytes;
          E.v = (const char *)E.v + (int64_t)l * s->layer_bytes;
        }
        pl->small_links[(size_t)l * nl + i] = E;
      }
  }
  const size_t tables = pl->small ? 0 : pl->table_bytes * s->n_layers;
  const size_t bytes = pl->small ? pl->C.part_bytes : tables + pl->C.work_bytes();
  if (bytes > 0) {
    DeviceGuard dg(s->device);
    if (!dg.ok) {
      delete pl;
      return fail(PIC_ERR_HIP, "cannot select the store's device");
    }
    hipError_t e = hipMalloc(&pl->dev, bytes);
    if (e != hipSuccess) {
      delete pl;
      return hip_fail(e, "hipMalloc(plan)");
    }
    pl->work = (char *)pl->dev + tables;
  }
  if (bytes > 0 && !pl->small) {
    DeviceGuard dg(s->device);
    if (!dg.ok) {
      (void)hipFree(pl->dev);
      delete pl;
      return fail(PIC_ERR_HIP, "cannot select the store's device");
    }
    // Every layer's tables differ only in the chunk links' addresses: layer
    // l of a slot sits l pool layers further on; own-KV links point at the
    // plan's workspace in every layer.
    std::vector<char> host(tables, 0);
    std::vector<LinkEntry> links(P.links);
    place_own(s, P, pl->work, links.data());
    std::vector<bool> own(nl, false);
    for (auto &o : P.own) own[o.first] = true;
    for (int32_t l = 0; l < s->n_layers; ++l) {
      std::vector<LinkEntry> at(links);
      for (size_t i = 0; i < nl; ++i)
        if (!own[i]) {
          at[i].k = (const char *)at[i].k + (int64_t)l * s->layer_bytes;
          at[i].v = (const char *)at[i].v + (int64_t)l * s->layer_bytes;
        }
      write_tables(pl->C, pl->layout, at.data(), host.data() + (size_t)l * pl->table_bytes);
    }
    hipError_t e = hipMemcpy(pl->dev, host.data(), tables, hipMemcpyHostToDevice);
    if (e != hipSuccess) {
      (void)hipFree(pl->dev);
      delete pl;
      return hip_fail(e, "hipMemcpy(plan tables)");
    }
  }
  for (uint64_t id : P.ids) ++s->map.at(id).plan_refs;
  ++s->live_plans;
  *out = pl;
  return PIC_OK;
}

pic_status pic_link_plan_run(pic_link_plan *pl, int32_t layer, const void *q, const void *k_self,
                             const void *v_self, float softmax_scale, void *out, float *lse,
                             void *stream) {
  if (!pl) return fail(PIC_ERR_INVALID, "plan is NULL");
  pic_store *s = pl->store;
  if (layer < 0 || layer >= s->n_layers)
    return fail(PIC_ERR_INVALID, "layer %d outside the store's %d layers", layer, s->n_layers);
  if (!std::isfinite(softmax_scale) || !(softmax_scale > 0.f))
    return fail(PIC_ERR_INVALID, "softmax_scale must be positive and finite");
  if (pl->batch == 0) return PIC_OK;
  pic_status rc = check_tensors(s, pl->C.P, q, k_self, v_self, out);
  if (rc != PIC_OK) return rc;
  if (pl->C.P.total_q == 0) return PIC_OK;
  DeviceGuard dg(s->device);
  if (!dg.ok) return fail(PIC_ERR_HIP, "cannot select the store's device");
  if (pl->small)
    return launch_small(s->desc, pl->C,
                        pl->small_links.data() + (size_t)layer * pl->C.P.links.size(),
                        pl->work, q, k_self, v_self, softmax_scale, out, lse,
                        (hipStream_t)stream);
  LinkParams lp = pl->C.lp;
  const char *t = (const char *)pl->dev + (size_t)layer * pl->table_bytes;
  point_tables(pl->C, pl->layout, t, lp);
  Prologue pro;
  pro.links = lp.links;
  pro.reqs = lp.reqs;
  return launch_call(s, pl->C, lp, pl->work, pro, q, k_self, v_self, softmax_scale, out, lse,
                     (hipStream_t)stream);
}

pic_status pic_link_plan_destroy(pic_link_plan *pl) {
  if (!pl) return PIC_OK;
  if (pl->dev) {
    DeviceGuard dg(pl->store->device);
    (void)hipDeviceSynchronize();
    (void)hipFree(pl->dev);
  }
  for (uint64_t id : pl->C.P.ids) {
    auto it = pl->store->map.find(id);
    if (it != pl->store->map.end()) --it->second.plan_refs;
  }
  --pl->store->live_plans;
  delete pl;
  return PIC_OK;
}

pic_status pic_debug_gather(pic_store *s, const uint64_t *ids, int32_t n, int32_t layer,
                            void *k_out, void *v_out, void *stream) {
  if (!s) return fail(PIC_ERR_INVALID, "store is NULL");
  if (n < 0 || (n > 0 && !ids)) return fail(PIC_ERR_INVALID, "bad id list");
  if (layer < 0 || layer >= s->n_layers)
    return fail(PIC_ERR_INVALID, "layer %d outside the store's %d layers", layer, s->n_layers);
  const bool gqa = s->desc.kind == PIC_GQA;
  std::vector<LinkEntry> links;
  links.reserve(n);
  int64_t toks = 0;
  for (int32_t i = 0; i < n; ++i) {
    auto it = s->map.find(ids[i]);
    if (it == s->map.end()) return fail(PIC_ERR_NOT_FOUND, "chunk id 0x%llx not in the store",
                                        (unsigned long long)ids[i]);
    for (const Run &r : it->second.runs) {
      LinkEntry E = run_entry(s, r, layer);
      E.tile0 = 0;
      E.tok0 = (int32_t)toks;
      links.push_back(E);
      toks += r.ntok;
    }
  }
  n = (int32_t)links.size();
  if (toks == 0) return PIC_OK;
  if (!k_out || (gqa && !v_out)) return fail(PIC_ERR_INVALID, "k_out/v_out is NULL");
  if (!gqa && v_out) return fail(PIC_ERR_INVALID, "v_out must be NULL for MLA");
  DeviceGuard dg(s->device);
  if (!dg.ok) return fail(PIC_ERR_HIP, "cannot select the store's device");
  const hipStream_t st = (hipStream_t)stream;
  Stage *stage = nullptr;
  pic_status rc = stage_acquire(s, sizeof(LinkEntry) * n, &stage);
  if (rc != PIC_OK) return rc;
  memcpy(stage->host, links.data(), sizeof(LinkEntry) * n);
  HIP_TRY(launch_table_copy(stage->host_dev, stage->dev, (int64_t)(sizeof(LinkEntry) * n), st),
          "table_copy_kernel");
  const pic_store_desc &d = s->desc;
  hipError_t e = launch_gather((const LinkEntry *)stage->dev, n, toks, d.n_kv_heads,
                               d.d_k, d.d_v, !gqa, s->esz, k_out, v_out, st);
  if (e != hipSuccess) return hip_fail(e, "gather_kernel");
  HIP_TRY(hipEventRecord(stage->done, st), "hipEventRecord(stage)");
  stage->pending = true;
  return PIC_OK;
}

pic_status pic_debug_request_order(const int32_t *q_len, const int32_t *self_len,
                                   const int32_t *doc_tiles, int32_t batch, int32_t n_q_heads,
                                   int32_t n_kv_heads, int32_t cus, int32_t xcds,
                                   int32_t *order_out, double *finish_out) {
  if (batch < 0 || (batch > 0 && (!q_len || !self_len || !doc_tiles || !order_out)))
    return fail(PIC_ERR_INVALID, "NULL array");
  if (n_kv_heads <= 0 || n_q_heads <= 0 || n_q_heads % n_kv_heads || cus <= 0 || xcds <= 0 ||
      cus % xcds)
    return fail(PIC_ERR_INVALID, "bad head counts or device shape");
  Plan P;
  P.reqs.resize(batch);
  int32_t max_rows = 0;
  const int group = n_q_heads / n_kv_heads;
  for (int32_t r = 0; r < batch; ++r) {
    if (q_len[r] < 0 || self_len[r] < 0 || doc_tiles[r] < 0 ||
        (int64_t)q_len[r] * group > INT32_MAX / 2 || self_len[r] > INT32_MAX / 2 ||
        doc_tiles[r] > INT32_MAX / 4)
      return fail(PIC_ERR_INVALID, "request %d: length out of range", r);
    ReqEntry &R = P.reqs[r];
    R = ReqEntry{};
    R.lq = q_len[r];
    R.ls = self_len[r];
    R.doc_tiles = doc_tiles[r];
    R.tiles = R.doc_tiles + (R.ls + kTile - 1) / kTile;
    max_rows = std::max(max_rows, R.lq * group);
  }
  // heaviest first, as plan_call orders
  P.order.resize(batch);
  for (int32_t r = 0; r < batch; ++r) P.order[r] = r;
  std::stable_sort(P.order.begin(), P.order.end(), [&](int32_t a, int32_t b) {
    return (int64_t)P.reqs[a].tiles * P.reqs[a].lq > (int64_t)P.reqs[b].tiles * P.reqs[b].lq;
  });
  LinkParams lp{};
  lp.batch = batch;
  lp.n_q_heads = n_q_heads;
  lp.n_kv_heads = n_kv_heads;
  lp.group = group;
  lp.n_xcd = xcds;
  const int rows_per_block = mfma_d128_rows_per_block();
  lp.nrb = std::max(1, (max_rows + rows_per_block - 1) / rows_per_block);
  lp.n_groups = (int32_t)round_up((int64_t)batch * n_kv_heads, xcds);
  double finish[2];
  balance_order_d128(nullptr, P, lp, rows_per_block, cus / xcds * mfma_d128_blocks_per_cu(), finish);
  std::copy(P.order.begin(), P.order.end(), order_out);
  if (finish_out) {
    finish_out[0] = finish[0];
    finish_out[1] = finish[1];
  }
  return PIC_OK;
}

namespace {

// Shared checks of the two MLA projections: sizes, 16-byte aligned device
// buffers.
pic_status check_proj(int32_t n_tokens, int32_t n_heads, std::initializer_list<const void *> bufs) {
  if (n_tokens < 0 || n_heads <= 0 || n_heads > 1024)
    return fail(PIC_ERR_INVALID, "n_tokens must be >= 0 and n_heads 1..1024");
  if ((int64_t)n_tokens * n_heads > INT32_MAX / 4) return fail(PIC_ERR_INVALID, "too many rows");
  if (n_tokens == 0) return PIC_OK;
  for (const void *b : bufs) {
    if (!b) return fail(PIC_ERR_INVALID, "a tensor pointer is NULL");
    if ((uintptr_t)b % 16) return fail(PIC_ERR_INVALID, "tensors must be 16-byte aligned");
  }
  return PIC_OK;
}

}  // namespace

pic_status pic_mla_absorb_q(int32_t n_tokens, int32_t n_heads, const void *q, const void *w_uk_t,
                            void *q_out, void *stream) {
  pic_status rc = check_proj(n_tokens, n_heads, {q, w_uk_t, q_out});
  if (rc != PIC_OK || n_tokens == 0) return rc;
  hipError_t e = launch_mla_absorb_q(q, w_uk_t, q_out, n_tokens, n_heads, device_shape(),
                                     (hipStream_t)stream);
  if (e != hipSuccess) return hip_fail(e, "proj_kernel (absorb)");
  return PIC_OK;
}

pic_status pic_mla_up_v(int32_t n_tokens, int32_t n_heads, const void *o_lat, const void *w_uv,
                        void *out, void *stream) {
  pic_status rc = check_proj(n_tokens, n_heads, {o_lat, w_uv, out});
  if (rc != PIC_OK || n_tokens == 0) return rc;
  hipError_t e = launch_mla_up_v(o_lat, w_uv, out, n_tokens, n_heads, device_shape(),
                                 (hipStream_t)stream);
  if (e != hipSuccess) return hip_fail(e, "proj_kernel (up)");
  return PIC_OK;
}

pic_status pic_prof_begin_sampled(int32_t every) {
  if (every < 1 || every > 1000000) return fail(PIC_ERR_INVALID, "every must be 1..1000000");
  std::lock_guard<std::mutex> g(g_prof.mu);
  for (auto &ev : g_prof.events) g_prof.spare.push_back(ev);
  g_prof.events.clear();
  g_prof.every = every;
  g_prof.seen = 0;
  g_prof.on = true;
  return PIC_OK;
}

pic_status pic_prof_begin(void) { return pic_prof_begin_sampled(1); }

pic_status pic_prof_end(double *kernel_ms, int64_t *launches, char *name_buf, int32_t name_len) {
  std::lock_guard<std::mutex> g(g_prof.mu);
  g_prof.on = false;
  double total = 0.0;
  for (auto &ev : g_prof.events) {
    HIP_TRY(hipEventSynchronize(ev.second), "hipEventSynchronize(prof)");
    float ms = 0.f;
    HIP_TRY(hipEventElapsedTime(&ms, ev.first, ev.second), "hipEventElapsedTime");
    total += ms;
  }
  if (kernel_ms) *kernel_ms = total;
  if (launches) *launches = (int64_t)g_prof.events.size();
  if (name_buf && name_len > 0) {
    snprintf(name_buf, (size_t)name_len, "%s", g_prof.name.c_str());
  }
  for (auto &ev : g_prof.events) g_prof.spare.push_back(ev);
  g_prof.events.clear();
  return PIC_OK;
}

// Times one launch of a peak microbenchmark on `stream` (blocking).
static pic_status time_peak(hipStream_t st, double *ms_out,
                            const std::function<hipError_t(float *)> &launch) {
  float *scratch = nullptr;
  HIP_TRY(hipMalloc(&scratch, (size_t)pic::peak_out_floats() * sizeof(float)), "hipMalloc(peak)");
  hipEvent_t e0 = nullptr, e1 = nullptr;
  hipError_t e = hipEventCreateWithFlags(&e0, hipEventDisableSystemFence);
  if (e == hipSuccess) e = hipEventCreateWithFlags(&e1, hipEventDisableSystemFence);
  if (e == hipSuccess) e = hipEventRecord(e0, st);
  if (e == hipSuccess) e = launch(scratch);
  if (e == hipSuccess) e = hipEventRecord(e1, st);
  if (e == hipSuccess) e = hipEventSynchronize(e1);
  float ms = 0.f;
  if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
  if (e0) (void)hipEventDestroy(e0);
  if (e1) (void)hipEventDestroy(e1);
  (void)hipFree(scratch);
  if (e != hipSuccess) return hip_fail(e, "peak microbenchmark");
  *ms_out = ms;
  return PIC_OK;
}

pic_status pic_peak_mfma_bf16(int32_t iters, double *tflops, void *stream) {
  if (!tflops) return fail(PIC_ERR_INVALID, "tflops is NULL");
  if (iters <= 0 || iters > (1 << 22)) return fail(PIC_ERR_INVALID, "iters must be 1..2^22");
  double ms = 0.0;
  const pic_status rc = time_peak((hipStream_t)stream, &ms, [&](float *out) {
    return pic::launch_peak_mfma(out, iters, (hipStream_t)stream);
  });
  if (rc != PIC_OK) return rc;
  *tflops = ms > 0.0 ? pic::peak_mfma_flops(iters) / (ms * 1e-3) / 1e12 : 0.0;
  return PIC_OK;
}

pic_status pic_peak_hbm_read(const void *buf, int64_t bytes, double *gbs, void *stream) {
  if (!gbs || !buf) return fail(PIC_ERR_INVALID, "buf and gbs must not be NULL");
  if (bytes <= 0 || bytes % 16 != 0 || (uintptr_t)buf % 16 != 0)
    return fail(PIC_ERR_INVALID, "bytes must be a positive multiple of 16 and buf 16-byte aligned");
  hipPointerAttribute_t at{};
  if (hipPointerGetAttributes(&at, buf) != hipSuccess || at.type != hipMemoryTypeDevice) {
    (void)hipGetLastError();
    return fail(PIC_ERR_INVALID, "buf is not device memory");
  }
  double ms = 0.0;
  const pic_status rc = time_peak((hipStream_t)stream, &ms, [&](float *out) {
    return pic::launch_peak_read(buf, bytes, out, (hipStream_t)stream);
  });
  if (rc != PIC_OK) return rc;
  *gbs = ms > 0.0 ? (double)bytes / (ms * 1e-3) / 1e9 : 0.0;
  return PIC_OK;
}

pic_status pic_peak_hbm_write(void *buf, int64_t bytes, double *gbs, void *stream) {
  if (!gbs || !buf) return fail(PIC_ERR_INVALID, "buf and gbs must not be NULL");
  if (bytes <= 0 || bytes % 16 != 0 || (uintptr_t)buf % 16 != 0)
    return fail(PIC_ERR_INVALID, "bytes must be a positive multiple of 16 and buf 16-byte aligned");
  hipPointerAttribute_t at{};
  if (hipPointerGetAttributes(&at, buf) != hipSuccess || at.type != hipMemoryTypeDevice) {
    (void)hipGetLastError();
    return fail(PIC_ERR_INVALID, "buf is not device memory");
  }
  double ms = 0.0;
  const pic_status rc = time_peak((hipStream_t)stream, &ms, [&](float *) {
    return pic::launch_peak_write(buf, bytes, (hipStream_t)stream);
  });
  if (rc != PIC_OK) return rc;
  *gbs = ms > 0.0 ? (double)bytes / (ms * 1e-3) / 1e9 : 0.0;
  return PIC_OK;
}

const char *pic_status_str(pic_status st) {
  switch (st) {
    case PIC_OK: return "PIC_OK";
    case PIC_ERR_INVALID: return "PIC_ERR_INVALID";
    case PIC_ERR_NOT_FOUND: return "PIC_ERR_NOT_FOUND";
    case PIC_ERR_EXISTS: return "PIC_ERR_EXISTS";
    case PIC_ERR_OOM: return "PIC_ERR_OOM";
    case PIC_ERR_HIP: return "PIC_ERR_HIP";
    case PIC_ERR_UNSUPPORTED: return "PIC_ERR_UNSUPPORTED";
  }
  return "PIC_ERR_?";
}

const char *pic_last_error(void) { return g_err.c_str(); }

}  // extern "C"
