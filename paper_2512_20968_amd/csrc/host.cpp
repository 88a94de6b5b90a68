// Host side of the mesh_attn C ABI: argument validation, error text, the
// canonical block work list, workgroup ordering and kernel launches.
//
// The work list follows the causal rule of Section 3.7 (a key is visible to a
// query iff its global position is not larger) applied per (Q block, KV block)
// pair; see include/mesh_attn.h for the exact layout.

#include "mesh_attn.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <map>
#include <memory>
#include <mutex>
#include <string>
#include <vector>

#include "host_error.h"
#include "internal.h"
#include "plan.h"

using namespace mesh_attn;
using mesh_attn::plan::Slice;
using mesh_attn::plan::token_pos;

static_assert(MA_NOALLOC_SCRATCH_BYTES == kNoAllocScratchBytes &&
                  MA_NOALLOC_MAX_LIST == kNoAllocMaxList &&
                  MA_NOALLOC_MAX_QBLOCKS == kNoAllocMaxQBlocks,
              "public limits of the allocation-free forward");

namespace {
thread_local std::string g_last_error;
}  // namespace

namespace mesh_attn {
namespace host {

ma_status_t fail(ma_status_t st, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof(buf), fmt, ap);
  va_end(ap);
  g_last_error = buf;
  return st;
}

ma_status_t ok() {
  g_last_error.clear();
  return MA_OK;
}

}  // namespace host
}  // namespace mesh_attn

namespace {

using mesh_attn::host::fail;
using mesh_attn::host::ok;

ma_status_t hip_fail(hipError_t e, const char* what) {
  return fail(MA_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
}

bool aligned16(const void* p) {
  return (reinterpret_cast<uintptr_t>(p) & 15u) == 0;
}

ma_status_t check_list(const char* name, const int32_t* idx, int32_t n,
                       int32_t num_partitions) {
  if (n < 1) return fail(MA_ERR_INVALID_ARG, "%s: length %d < 1", name, n);
  if (!idx) return fail(MA_ERR_INVALID_ARG, "%s is NULL", name);
  std::vector<char> seen(static_cast<size_t>(num_partitions), 0);
  for (int32_t i = 0; i < n; ++i) {
    if (idx[i] < 0 || idx[i] >= num_partitions)
      return fail(MA_ERR_INVALID_ARG, "%s[%d] = %d outside [0, %d)", name, i,
                  idx[i], num_partitions);
    if (seen[idx[i]])
      return fail(MA_ERR_INVALID_ARG, "%s[%d] = %d is a duplicate", name, i,
                  idx[i]);
    seen[idx[i]] = 1;
  }
  return MA_OK;
}

ma_status_t check_problem(const ma_problem_t* p) {
  if (!p) return fail(MA_ERR_INVALID_ARG, "problem is NULL");
  if (p->num_partitions < 1)
    return fail(MA_ERR_INVALID_ARG, "num_partitions %d < 1", p->num_partitions);
  if (p->partition_len < 1)
    return fail(MA_ERR_INVALID_ARG, "partition_len %d < 1", p->partition_len);
  if (static_cast<int64_t>(p->num_partitions) * p->partition_len >
      (int64_t{1} << 30))
    return fail(MA_ERR_INVALID_ARG,
                "sequence of %lld tokens exceeds 2^30",
                static_cast<long long>(p->num_partitions) * p->partition_len);
  if (p->num_q_heads < 1 || p->num_kv_heads < 1)
    return fail(MA_ERR_INVALID_ARG, "head counts must be >= 1 (Hq %d, Hkv %d)",
                p->num_q_heads, p->num_kv_heads);
  if (p->num_q_heads % p->num_kv_heads != 0)
    return fail(MA_ERR_INVALID_ARG, "num_q_heads %d not a multiple of "
                "num_kv_heads %d", p->num_q_heads, p->num_kv_heads);
  if (p->causal != 0 && p->causal != 1)
    return fail(MA_ERR_INVALID_ARG, "causal must be 0 or 1, got %d", p->causal);
  if (p->layout != MA_LAYOUT_CONTIGUOUS && p->layout != MA_LAYOUT_STRIPED)
    return fail(MA_ERR_INVALID_ARG, "layout must be %d or %d, got %d",
                MA_LAYOUT_CONTIGUOUS, MA_LAYOUT_STRIPED, p->layout);
  if (!(p->softmax_scale > 0.f) || !std::isfinite(p->softmax_scale))
    return fail(MA_ERR_INVALID_ARG, "softmax_scale must be finite and > 0");
  if (p->head_dim < 1)
    return fail(MA_ERR_INVALID_ARG, "head_dim %d < 1", p->head_dim);
  return MA_OK;
}

ma_status_t check_blocks(const ma_problem_t* p, int32_t bm, int32_t bn) {
  if (bm < 1 || bn < 1)
    return fail(MA_ERR_INVALID_ARG, "block sizes must be >= 1 (%d, %d)", bm, bn);
  if (p->partition_len % bm != 0 || p->partition_len % bn != 0)
    return fail(MA_ERR_INVALID_ARG,
                "partition_len %d must be a multiple of the block sizes "
                "(%d, %d)", p->partition_len, bm, bn);
  return MA_OK;
}

ma_status_t check_tile(const ma_problem_t* p, const int32_t* q_idx, int32_t nq,
                       const int32_t* kv_idx, int32_t nkv) {
  ma_status_t st = check_problem(p);
  if (st != MA_OK) return st;
  st = check_list("q_idx", q_idx, nq, p->num_partitions);
  if (st != MA_OK) return st;
  return check_list("kv_idx", kv_idx, nkv, p->num_partitions);
}

// Class of one block pair from its extreme token positions.
inline int block_class(int64_t q_first, int64_t q_last, int64_t k_first,
                       int64_t k_last, bool causal) {
  if (!causal) return MA_CLS_FULL;
  if (k_first > q_last) return MA_CLS_EMPTY;   // every key after every query
  if (k_last <= q_first) return MA_CLS_FULL;   // every key at/before every query
  return MA_CLS_PARTIAL;
}

struct Run {
  int32_t row, list, begin, end, cls;
};

// Runs of one orientation.  "Rows" are the blocks of side A (bm_a rows each,
// lists a_idx), walked in buffer order; for each row, every list entry of side
// B (blocks of bm_b) yields maximal equal-class runs, EMPTY dropped.  When
// a_is_q, side A is the query side.  Each side's buffer holds slice sa / sb of
// each of its partitions.
void build_runs(const ma_problem_t* p, const int32_t* a_idx, int32_t na,
                int32_t bm_a, Slice sa, const int32_t* b_idx, int32_t nb,
                int32_t bm_b, Slice sb, bool a_is_q, std::vector<int32_t>* ptr,
                std::vector<Run>* runs) {
  const int32_t nab = static_cast<int32_t>(sa.len / bm_a);
  const int32_t nbb = static_cast<int32_t>(sb.len / bm_b);
  const bool causal = p->causal != 0;
  ptr->assign(static_cast<size_t>(na) * nab + 1, 0);
  runs->clear();
  for (int32_t a = 0; a < na; ++a) {
    for (int32_t ab = 0; ab < nab; ++ab) {
      const int32_t row = a * nab + ab;
      (*ptr)[row] = static_cast<int32_t>(runs->size());
      const int64_t a_row = sa.off + int64_t{ab} * bm_a;
      const int64_t a_first = token_pos(p, a_idx[a], a_row);
      const int64_t a_last = token_pos(p, a_idx[a], a_row + bm_a - 1);
      for (int32_t b = 0; b < nb; ++b) {
        int32_t kb = 0, cur = -1, start = 0;
        for (; kb <= nbb; ++kb) {
          int c = -2;
          if (kb < nbb) {
            const int64_t b_row = sb.off + int64_t{kb} * bm_b;
            const int64_t b_first = token_pos(p, b_idx[b], b_row);
            const int64_t b_last = token_pos(p, b_idx[b], b_row + bm_b - 1);
            c = a_is_q ? block_class(a_first, a_last, b_first, b_last, causal)
                       : block_class(b_first, b_last, a_first, a_last, causal);
          }
          if (c != cur) {
            if (cur > MA_CLS_EMPTY) runs->push_back({row, b, start, kb, cur});
            cur = c;
            start = kb;
          }
        }
      }
    }
  }
  (*ptr)[static_cast<size_t>(na) * nab] = static_cast<int32_t>(runs->size());
}

ma_status_t export_runs(const std::vector<int32_t>& ptr,
                        const std::vector<Run>& runs, int32_t* out_ptr,
                        ma_run_t* out_runs, int64_t cap, int64_t* n_runs) {
  if (n_runs) *n_runs = static_cast<int64_t>(runs.size());
  if (out_ptr) std::memcpy(out_ptr, ptr.data(), ptr.size() * sizeof(int32_t));
  if (static_cast<int64_t>(runs.size()) > cap || (!out_runs && !runs.empty()))
    return fail(MA_ERR_CAPACITY, "run list needs %zu entries, capacity %lld",
                runs.size(), static_cast<long long>(cap));
  for (size_t i = 0; i < runs.size(); ++i)
    out_runs[i] = ma_run_t{runs[i].row, runs[i].list, runs[i].begin,
                           runs[i].end, runs[i].cls};
  return ok();
}

// ---------------------------------------------------------------------------
// Device plans: the order table, runs and split rows of a call's passes
// (plan.h).  A list of at most kInlinePlan bytes is built on the stack for
// every call and travels in the kernel's arguments.  A longer one is packed
// into one pinned host buffer that a kernel copies to the caller's workspace
// on the caller's stream.
//
// The longer plans are cached per tile (at most kMaxPlans, least recently used
// evicted).  A pinned source must outlive every asynchronous copy from it, and
// freeing pinned memory would wait for the device, so buffers are never freed
// while the library is in use: every upload records an event on the caller's
// stream, an evicted plan's buffer joins a spare list, and a spare buffer is
// reused for a new plan only once all events recorded after copies from it
// have completed (hipEventQuery, which does not wait) and no call is between
// finding its plan and recording its event.  No call synchronizes.
// ---------------------------------------------------------------------------

constexpr size_t kAlign = 256;
inline size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

// One pass's lists within a plan's bytes.
struct PassView {
  size_t off_rows = 0, off_runs = 0, off_splits = 0, off_queue = 0;
  int32_t m = 0, n_items = 0, n_splits = 0, parts = 0, mode = 0;
  bool is_short = false;
};

// An event recorded after a copy, with the device it belongs to (an event
// can only be recorded on a stream of the device it was created on).
struct PendingEvent {
  hipEvent_t ev;
  int dev;
};

struct PinnedBuf {
  void* host = nullptr;
  size_t cap = 0;
  std::vector<PendingEvent> pending;  // recorded after copies from this buffer
  int in_use = 0;  // calls that have yet to record theirs, or could not
};

struct Plan {
  PinnedBuf* buf = nullptr;
  size_t bytes = 0;
  PassView a, b;         // fwd uses a; bwd uses a (Q-major) and b (KV-major)
  uint64_t last_use = 0;
};

// What the launches need from a plan: the workspace bytes it takes and its
// passes; src: the pinned copy, or null if the lists are in `blob`.
struct PlanView {
  size_t bytes = 0;
  PassView a, b;
  const void* src = nullptr;
};

std::mutex g_plan_mu;
std::map<std::string, Plan> g_plans;
std::vector<PinnedBuf*> g_spare;       // buffers of evicted plans
std::map<int, std::vector<hipEvent_t>> g_free_events;  // per device, completed
uint64_t g_plan_clock = 0;
constexpr size_t kMaxPlans = 1024;

// Drops the completed events of `b` (to the free list); true if none remain.
bool retire_completed(PinnedBuf* b) {
  size_t keep = 0;
  for (const PendingEvent& pe : b->pending) {
    if (hipEventQuery(pe.ev) == hipSuccess)
      g_free_events[pe.dev].push_back(pe.ev);
    else
      b->pending[keep++] = pe;
  }
  b->pending.resize(keep);
  return keep == 0;
}

// A pinned buffer of at least `bytes`: an idle spare if one is large enough
// (the smallest such), else a new allocation.
ma_status_t take_buffer(size_t bytes, PinnedBuf** out) {
  size_t best = g_spare.size();
  for (size_t i = 0; i < g_spare.size(); ++i) {
    PinnedBuf* b = g_spare[i];
    if (b->cap < bytes || b->in_use > 0 || !retire_completed(b)) continue;
    if (best == g_spare.size() || b->cap < g_spare[best]->cap) best = i;
  }
  if (best != g_spare.size()) {
    *out = g_spare[best];
    g_spare.erase(g_spare.begin() + best);
    return MA_OK;
  }
  auto* b = new PinnedBuf;
  b->cap = std::max(bytes, kAlign);
  // Read by kernels, on whichever device a call runs.
  hipError_t e = hipHostMalloc(&b->host, b->cap,
                               hipHostMallocPortable | hipHostMallocMapped);
  if (e != hipSuccess) {
    delete b;
    return hip_fail(e, "hipHostMalloc(work list)");
  }
  *out = b;
  return MA_OK;
}

// What a plan depends on: head_dim too, through the cut (the passes of
// internal.h) and fwd_is_short.
std::string plan_key(int pass, const ma_problem_t* p, const int32_t* q_idx,
                     int32_t nq, const int32_t* kv_idx, int32_t nkv,
                     const ma_chunk_t& ch) {
  std::string k;
  auto put = [&k](const void* d, size_t n) {
    k.append(static_cast<const char*>(d), n);
  };
  put(&pass, sizeof pass);
  put(&ch, sizeof ch);
  put(&p->num_partitions, sizeof(int32_t));
  put(&p->partition_len, sizeof(int32_t));
  put(&p->num_q_heads, sizeof(int32_t));
  put(&p->num_kv_heads, sizeof(int32_t));
  put(&p->head_dim, sizeof(int32_t));
  put(&p->causal, sizeof(int32_t));
  put(&p->layout, sizeof(int32_t));
  put(&nq, sizeof nq);
  put(q_idx, sizeof(int32_t) * nq);
  put(&nkv, sizeof nkv);
  put(kv_idx, sizeof(int32_t) * nkv);
  return k;
}

// Packs the lists of one built side behind `off`; returns the end.
size_t pack_side(const plan::Built& b, const plan::Arrays& arr, int32_t heads,
                 size_t align, char* base, size_t off, PassView* v) {
  auto put = [&](const void* src, size_t bytes) {
    const size_t at = off;
    if (bytes > 0) std::memcpy(base + at, src, bytes);
    off = (at + bytes + align - 1) / align * align;
    return at;
  };
  v->off_rows = put(arr.rows, b.m * sizeof(DevRow));
  v->off_runs = put(arr.runs, b.n_runs * sizeof(DevRun));
  v->off_splits = put(arr.splits, b.n_splits * sizeof(DevSplit));
  // The item counters, one per XCD lane (see queued_static_slots), zero.
  const int32_t zeros[kNumXcd] = {};
  v->off_queue = put(zeros, sizeof zeros);
  v->m = b.m;
  v->n_items = b.m * heads;
  v->n_splits = b.n_splits;
  v->parts = b.parts;
  v->mode = b.mode;
  v->is_short = b.is_short;
  return off;
}

// The order of a pass for its kernels, its lists at `base` (device), or in the
// PlanBlob if base is null.
DevOrder order_at(const PassView& v, char* base) {
  DevOrder o{};
  if (base) {
    o.rows = reinterpret_cast<const DevRow*>(base + v.off_rows);
    o.runs = reinterpret_cast<const DevRun*>(base + v.off_runs);
    o.splits = reinterpret_cast<const DevSplit*>(base + v.off_splits);
    o.queue = reinterpret_cast<int32_t*>(base + v.off_queue);
  } else {
    o.inline_list = 1;
    o.off_runs = static_cast<int32_t>(v.off_runs);
    o.off_splits = static_cast<int32_t>(v.off_splits);
  }
  o.m = v.m;
  o.n_items = v.n_items;
  o.mode = v.mode;
  o.parts = v.parts;
  o.n_splits = v.n_splits;
  o.is_short = v.is_short;
  return o;
}

// Builds one or two sides into `blob` without heap memory; false if they do
// not fit or take their last items from counters (which a PlanBlob, read in
// place, does not hold).
bool inline_plan(const plan::Side* sides, int n, PlanBlob* blob,
                 PlanView* view) {
  constexpr int kRows = kInlinePlan / sizeof(DevRow);
  constexpr int kRuns = kInlinePlan / sizeof(DevRun);
  constexpr int kSplits = kInlinePlan / sizeof(DevSplit);
  DevRow rows[kRows];
  DevRun runs[kRuns];
  DevSplit splits[kSplits];
  int32_t work[kRows];
  const plan::Arrays arr{rows, kRows, runs, kRuns, splits, kSplits, work};
  size_t off = 0;
  for (int i = 0; i < n; ++i) {
    plan::Built b;
    if (!plan::build(sides[i], arr, &b)) return false;
    if (int64_t{b.m} * sides[i].heads >= kQueuedMinItems) return false;
    const size_t need = b.m * sizeof(DevRow) + b.n_runs * sizeof(DevRun) +
                        b.n_splits * sizeof(DevSplit) + kNumXcd * 4 + 64;
    if (off + need > kInlinePlan) return false;
    off = pack_side(b, arr, sides[i].heads, 16, blob->bytes, off,
                    i == 0 ? &view->a : &view->b);
  }
  view->bytes = off;
  view->src = nullptr;
  return true;
}

// Whether the lists are likely too long for a PlanBlob, from sizes alone: an
// entry per row, or where items may be split about as many as fill the chip in
// one round, and the runs.  Such calls look in the cache before they build
// anything (a lookup takes 0.2 us, building a list up to its overflow 2 to 41
// us); a wrong guess costs that time and no more.
bool likely_long(const plan::Side* sides, int n) {
  int64_t bytes = 0;
  for (int i = 0; i < n; ++i) {
    const plan::Side& s = sides[i];
    const int64_t rows = s.rows(), items = rows * s.heads;
    const int64_t longest = s.nb * (s.sb.len / s.bm_b) * s.walks;
    int64_t entries = rows;
    if (s.pass && items <= s.pass->max_items &&
        longest > 2 * s.pass->min_piece &&
        !(s.forward &&
          fwd_is_short(items, static_cast<int32_t>(longest), s.p->head_dim)))
      entries = std::max<int64_t>(rows, s.pass->slots / s.heads);
    const int64_t runs = !s.p->causal                          ? 1
                         : s.p->layout == MA_LAYOUT_CONTIGUOUS ? 2
                                                               : 2 * s.nb;
    bytes += entries * sizeof(DevRow) + rows * runs * sizeof(DevRun);
  }
  return bytes > kInlinePlan;
}

// Upper bound of one side's packed bytes from sizes alone (at most two
// non-empty runs per (block, list entry): along a partition visibility only
// drops, FULL blocks first, then PARTIAL, then EMPTY).
size_t side_bound(int64_t n_blocks, int64_t n_list) {
  return align_up(n_blocks * sizeof(DevRow)) +
         align_up(n_blocks * n_list * 2 * sizeof(DevRun)) +
         align_up(kNumXcd * 4);
}

// What the allocation-free forward is limited by: 4 bytes per Q block, 8 per item
// and two runs per Q block and KV partition.  An upper bound of no list that is
// built today (its runs are the largest part of the device-built one, whose
// table lies beside the scratch array); kept as the public limit, so that every
// tile that was served is.
size_t noalloc_list_bytes(int64_t n_blocks, int64_t n_list, int64_t heads) {
  return align_up((n_blocks + 1) * 4) +
         align_up(n_blocks * n_list * 2 * sizeof(DevRun)) +
         align_up((n_blocks * heads + kNumXcd) * 8) + align_up(kNumXcd * 4);
}

// What splitting adds to one side: table entries of the pieces, the split rows
// (per head, so never more than the partials), and `parts` partial results of
// part_bytes.
size_t split_bound(int64_t parts, size_t part_bytes) {
  if (parts == 0) return 0;
  return align_up(parts * sizeof(DevRow)) +
         align_up(parts * sizeof(DevSplit)) + align_up(parts * part_bytes);
}

constexpr ma_chunk_t kWholeTile{0, 1, 0, 1};

// Partial results of a plan against the slots that the call has room for.
ma_status_t check_parts(const PassView& v, int32_t heads, int64_t slots) {
  if (int64_t{v.parts} * heads <= slots) return MA_OK;
  return fail(MA_ERR_WORKSPACE_TOO_SMALL,
              "work list of %d partial results for each of %d heads, room for "
              "%lld", v.parts, heads, static_cast<long long>(slots));
}

// The sides of a call: the forward's Q-major one, or the backward's Q-major
// (dQ) and KV-major (dK/dV) ones.  Returns their number.
int sides_of(int pass, const ma_problem_t* p, const int32_t* q_idx, int32_t nq,
             const int32_t* kv_idx, int32_t nkv, const ma_chunk_t& ch,
             bool may_split, plan::Side out[2]) {
  const int64_t P = p->partition_len;
  const Slice sq{P / ch.num_q_chunks, ch.q_chunk * (P / ch.num_q_chunks)};
  const Slice skv{P / ch.num_kv_chunks, ch.kv_chunk * (P / ch.num_kv_chunks)};
  const int32_t g = p->num_q_heads / p->num_kv_heads;
  auto may = [&](const split::Pass& ps) { return may_split ? &ps : nullptr; };
  if (pass == 0) {
    out[0] = plan::Side{p,   q_idx, nq,   kFwdBM, sq, kv_idx, nkv, kFwdBN,
                        skv, true,  p->num_q_heads, g, 1, may(fwd_pass(p->head_dim)), true};
    return 1;
  }
  out[0] = plan::Side{p,   q_idx, nq,   kBwdBM, sq, kv_idx, nkv, kBwdBN,
                      skv, true,  p->num_q_heads, g, 1, may(dq_pass(p->head_dim)), false};
  out[1] = plan::Side{p,  kv_idx, nkv,  kBwdBN, skv, q_idx, nq, kBwdBM,
                      sq, false,  p->num_kv_heads, 1, g, may(dkdv_pass(p->head_dim)), false};
  return 2;
}

// The cached plan of a call, built into a pinned buffer if it is not there.
// Called with the cache locked.
ma_status_t cached_plan(const std::string& key, const plan::Side* sides, int n,
                        Plan** out) {
  auto it = g_plans.find(key);
  if (it == g_plans.end()) {
    std::vector<char> bytes;
    Plan made;
    for (int i = 0; i < n; ++i) {
      const plan::Side& s = sides[i];
      const int64_t rows = s.rows();
      const int64_t extra = s.pass ? s.pass->max_parts() : 0;
      std::vector<DevRow> table(rows + extra);
      std::vector<DevRun> runs(rows * s.nb * 2);
      std::vector<DevSplit> splits(extra);
      std::vector<int32_t> work(rows);
      const plan::Arrays arr{table.data(),  rows + extra,
                             runs.data(),   static_cast<int64_t>(runs.size()),
                             splits.data(), extra, work.data()};
      plan::Built b;
      if (!plan::build(s, arr, &b))
        return fail(MA_ERR_CAPACITY, "work list of %lld rows",
                    static_cast<long long>(rows));
      bytes.resize(bytes.size() + align_up(b.m * sizeof(DevRow)) +
                   align_up(b.n_runs * sizeof(DevRun)) +
                   align_up(b.n_splits * sizeof(DevSplit)) +
                   align_up(kNumXcd * 4));
      made.bytes = pack_side(b, arr, s.heads, kAlign, bytes.data(), made.bytes,
                             i == 0 ? &made.a : &made.b);
    }
    if (g_plans.size() >= kMaxPlans) {
      auto lru = g_plans.begin();
      for (auto i = g_plans.begin(); i != g_plans.end(); ++i)
        if (i->second.last_use < lru->second.last_use) lru = i;
      g_spare.push_back(lru->second.buf);
      g_plans.erase(lru);
    }
    ma_status_t st = take_buffer(made.bytes, &made.buf);
    if (st != MA_OK) return st;
    std::memcpy(made.buf->host, bytes.data(), made.bytes);
    it = g_plans.emplace(key, made).first;
  }
  it->second.last_use = ++g_plan_clock;
  *out = &it->second;
  return MA_OK;
}

// Runs `launch(view)`, which enqueues the work of a call on `stream`, with the
// call's plan in `blob` or in a pinned buffer.  A pinned one is marked in use
// until the event behind that work is recorded, so that no other thread can
// recycle it in between; the cache is not locked meanwhile (a launch may wait
// for room in its queue).
template <class F>
ma_status_t with_plan(int pass, const ma_problem_t* p, const int32_t* q_idx,
                      int32_t nq, const int32_t* kv_idx, int32_t nkv,
                      const ma_chunk_t& ch, bool may_split, hipStream_t stream,
                      PlanBlob* blob, F&& launch) {
  plan::Side sides[2];
  const int n =
      sides_of(pass, p, q_idx, nq, kv_idx, nkv, ch, may_split, sides);
  PlanView view;
  const bool cache_first = likely_long(sides, n);
  if (!cache_first && inline_plan(sides, n, blob, &view)) return launch(view);
  const std::string key =
      plan_key(pass * 2 + may_split, p, q_idx, nq, kv_idx, nkv, ch);
  PinnedBuf* buf = nullptr;
  PendingEvent pe{nullptr, 0};
  {
    std::unique_lock<std::mutex> lock(g_plan_mu);
    if (cache_first && g_plans.find(key) == g_plans.end()) {
      lock.unlock();
      if (inline_plan(sides, n, blob, &view)) return launch(view);
      lock.lock();
    }
    Plan* plan = nullptr;
    const ma_status_t st = cached_plan(key, sides, n, &plan);
    if (st != MA_OK) return st;
    buf = plan->buf;
    retire_completed(buf);  // keeps the list as short as the copies in flight
    hipError_t e = hipGetDevice(&pe.dev);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    std::vector<hipEvent_t>& pool = g_free_events[pe.dev];
    if (!pool.empty()) {
      pe.ev = pool.back();
      pool.pop_back();
    } else {
      e = hipEventCreateWithFlags(&pe.ev, hipEventDisableTiming |
                                              hipEventDisableSystemFence);
      if (e != hipSuccess) return hip_fail(e, "hipEventCreateWithFlags");
    }
    view.bytes = plan->bytes;
    view.a = plan->a;
    view.b = plan->b;
    view.src = buf->host;
    ++buf->in_use;
  }
  const ma_status_t st = launch(view);
  // Also after a failed launch: the copy may have been enqueued before it.
  const hipError_t e = hipEventRecord(pe.ev, stream);
  std::lock_guard<std::mutex> lock(g_plan_mu);
  if (e != hipSuccess) {
    // The work is on its way, so the call has not failed; but nothing will
    // tell when the list has been read: the buffer stays in use for good.
    (void)hipGetLastError();  // or the next launch would report it
    g_free_events[pe.dev].push_back(pe.ev);
    return st;
  }
  buf->pending.push_back(pe);
  --buf->in_use;
  return st;
}

size_t fwd_ws_bound(const ma_problem_t* p, int32_t nq, int32_t nkv) {
  const int64_t nqb = int64_t{nq} * p->partition_len / kFwdBM;
  return side_bound(nqb, nkv);
}

size_t fwd_part_bytes(const ma_problem_t* p) {
  return static_cast<size_t>(kFwdBM) * (p->head_dim + 1) * 4;
}

// What splitting the forward's items adds to fwd_ws_bound: for this chunk pair
// alone, or (smaller_too) also for every tile of fewer partitions and every
// chunk pair of them.  Those have no more blocks, but may be split where this
// one has too many items.
size_t fwd_split_bytes(const ma_problem_t* p, int32_t nq, int32_t nkv,
                       const ma_chunk_t& ch, bool smaller_too) {
  const int64_t P = p->partition_len;
  const int64_t items = nq * (P / ch.num_q_chunks / kFwdBM) * p->num_q_heads;
  const int64_t blocks = nkv * (P / ch.num_kv_chunks / kFwdBN);
  const split::Pass& ps = fwd_pass(p->head_dim);
  const int64_t counted =
      smaller_too ? std::min<int64_t>(items, ps.max_items) : items;
  const int64_t parts = split::parts_bound(counted, blocks, ps);
  return split_bound(parts, fwd_part_bytes(p));
}

size_t bwd_ws_bound(const ma_problem_t* p, int32_t nq, int32_t nkv) {
  const int64_t nqb = int64_t{nq} * p->partition_len / kBwdBM;
  const int64_t nkb = int64_t{nkv} * p->partition_len / kBwdBN;
  const int64_t rows_q = int64_t{nq} * p->partition_len;
  return side_bound(nqb, nkv) + side_bound(nkb, nq) +
         2 * align_up(static_cast<size_t>(rows_q) * p->num_q_heads * 4);
}

// Partial slots of the split backward passes, and what splitting adds to
// bwd_ws_bound (smaller_too as in fwd_split_bytes).
struct BwdParts {
  int64_t kv, q;
  size_t kv_bytes, q_bytes;  // of the partial results
  size_t bytes;
};

BwdParts bwd_parts(const ma_problem_t* p, int32_t nq, int32_t nkv,
                   const ma_chunk_t& ch, bool smaller_too) {
  const int64_t P = p->partition_len;
  const int64_t nqb = nq * (P / ch.num_q_chunks / kBwdBM);
  const int64_t nkb = nkv * (P / ch.num_kv_chunks / kBwdBN);
  const int64_t kv_items = nkb * p->num_kv_heads;
  const int64_t q_items = nqb * p->num_q_heads;
  auto parts = [&](int64_t items, int64_t blocks, const split::Pass& ps) {
    return split::parts_bound(
        smaller_too ? std::min<int64_t>(items, ps.max_items) : items, blocks,
        ps);
  };
  const int32_t g = p->num_q_heads / p->num_kv_heads;
  BwdParts b{parts(kv_items, nqb * g, dkdv_pass(p->head_dim)),
             parts(q_items, nkb, dq_pass(p->head_dim)), 0, 0, 0};
  const size_t tile = size_t{128} * p->head_dim * 4;
  static_assert(kBwdBM == 128 && kBwdBN == 128, "rows of a partial result");
  b.kv_bytes = align_up(b.kv * 2 * tile);
  b.q_bytes = align_up(b.q * tile);
  b.bytes = split_bound(b.kv, 2 * tile) + split_bound(b.q, tile);
  return b;
}

ma_status_t check_head_dim(const ma_problem_t* p) {
  if (p->head_dim != 64 && p->head_dim != 128)
    return fail(MA_ERR_UNSUPPORTED, "head_dim %d unsupported (64 or 128)",
                p->head_dim);
  return MA_OK;
}

constexpr float kLog2e = 1.4426950408889634f;

ma_status_t check_chunk(const ma_problem_t* p, const ma_chunk_t& c, int32_t bm,
                        int32_t bn) {
  if (c.num_q_chunks < 1 || c.num_kv_chunks < 1)
    return fail(MA_ERR_INVALID_ARG, "chunk counts must be >= 1 (%d, %d)",
                c.num_q_chunks, c.num_kv_chunks);
  if (c.q_chunk < 0 || c.q_chunk >= c.num_q_chunks || c.kv_chunk < 0 ||
      c.kv_chunk >= c.num_kv_chunks)
    return fail(MA_ERR_INVALID_ARG, "chunk (%d of %d, %d of %d) out of range",
                c.q_chunk, c.num_q_chunks, c.kv_chunk, c.num_kv_chunks);
  const int64_t P = p->partition_len;
  if (P % c.num_q_chunks != 0 || (P / c.num_q_chunks) % bm != 0 ||
      P % c.num_kv_chunks != 0 || (P / c.num_kv_chunks) % bn != 0)
    return fail(MA_ERR_INVALID_ARG,
                "partition_len %lld must split into %d Q chunks of whole "
                "%d-row blocks and %d KV chunks of whole %d-row blocks",
                static_cast<long long>(P), c.num_q_chunks, bm,
                c.num_kv_chunks, bn);
  return MA_OK;
}

// Partial slots of a split forward.
int64_t parts_of(const ma_problem_t* p, int32_t nq, int32_t nkv,
                 const ma_chunk_t& ch) {
  const int64_t P = p->partition_len;
  return split::parts_bound(
      nq * (P / ch.num_q_chunks / kFwdBM) * p->num_q_heads,
      nkv * (P / ch.num_kv_chunks / kFwdBN), fwd_pass(p->head_dim));
}

// KV blocks that Q block `qb` of a whole tile sees (its work), without a run
// list: along a partition the visible blocks are a prefix.
int32_t visible_blocks(const ma_problem_t* p, const int32_t* q_idx,
                       const int32_t* kv_idx, int32_t nkv, int64_t qb) {
  const int64_t P = p->partition_len, qpb = P / kFwdBM, nbb = P / kFwdBN;
  if (!p->causal) return static_cast<int32_t>(nkv * nbb);
  const int64_t q_last =
      token_pos(p, q_idx[qb / qpb], (qb % qpb) * kFwdBM + kFwdBM - 1);
  const int64_t step = token_pos(p, 0, kFwdBN);  // positions per KV block
  int64_t n = 0;
  for (int32_t b = 0; b < nkv; ++b)
    n += plan::count_le(token_pos(p, kv_idx[b], 0), step, q_last, nbb);
  return static_cast<int32_t>(n);
}

// The cut of a tile for the device-side list builder, the pieces and split
// rows of one head.  Uses no heap.
struct NoAllocSplit {
  split::Cut cut;
  int32_t row_pieces, split_rows, parts;
  bool is_short;
};

NoAllocSplit noalloc_split(const ma_problem_t* p, const int32_t* q_idx,
                           int32_t nq, const int32_t* kv_idx, int32_t nkv) {
  int32_t work[kSplitMaxRows];
  const int32_t nqb =
      static_cast<int32_t>(int64_t{nq} * p->partition_len / kFwdBM);
  for (int32_t qb = 0; qb < nqb; ++qb)
    work[qb] = visible_blocks(p, q_idx, kv_idx, nkv, qb);
  NoAllocSplit s{{}, 0, 0, 0, false};
  s.is_short = fwd_is_short(int64_t{nqb} * p->num_q_heads,
                            *std::max_element(work, work + nqb), p->head_dim);
  if (!s.is_short)
    s.cut = split::choose(work, nqb, p->num_q_heads, fwd_pass(p->head_dim));
  if (s.cut.c == 0) return s;
  for (int32_t qb = 0; qb < nqb; ++qb) {
    const int32_t n = split::num_pieces(s.cut, qb, work[qb]);
    s.row_pieces += n;
    if (n == 1) continue;
    ++s.split_rows;
    s.parts += n;
  }
  return s;
}

// Forward of one chunk pair of a tile (the whole tile: one chunk each).
ma_status_t fwd_impl(const ma_problem_t* prob, const int32_t* q_idx,
                     int32_t nq, const int32_t* kv_idx, int32_t nkv,
                     const ma_chunk_t& ch, const void* q, const void* k,
                     const void* v, void* o, bool o_f32, float* lse,
                     int32_t accumulate, void* ws, size_t ws_bytes,
                     hipStream_t stream) {
  ma_status_t st = check_tile(prob, q_idx, nq, kv_idx, nkv);
  if (st == MA_OK) st = check_head_dim(prob);
  if (st == MA_OK) st = check_blocks(prob, kFwdBM, kFwdBN);
  if (st == MA_OK) st = check_chunk(prob, ch, kFwdBM, kFwdBN);
  if (st != MA_OK) return st;
  const void* ptrs[] = {q, k, v, o, lse, ws};
  const char* names[] = {"q", "k", "v", "o", "lse", "ws"};
  for (int i = 0; i < 6; ++i) {
    if (!ptrs[i]) return fail(MA_ERR_INVALID_ARG, "%s is NULL", names[i]);
    if (!aligned16(ptrs[i]))
      return fail(MA_ERR_INVALID_ARG, "%s is not 16-byte aligned", names[i]);
  }
  const size_t need = fwd_ws_bound(prob, nq, nkv);
  if (ws_bytes < need)
    return fail(MA_ERR_WORKSPACE_TOO_SMALL, "workspace %zu bytes < %zu",
                ws_bytes, need);
  // A workspace without room for partial results serves the call with whole
  // items.
  const bool may_split =
      ws_bytes >= need + fwd_split_bytes(prob, nq, nkv, ch, false);
  char* wsb = static_cast<char*>(ws);
  FwdParams fp{};
  fp.q = static_cast<const uint16_t*>(q);
  fp.k = static_cast<const uint16_t*>(k);
  fp.v = static_cast<const uint16_t*>(v);
  fp.o = o;
  fp.lse = lse;
  fp.rows_q = int64_t{nq} * (prob->partition_len / ch.num_q_chunks);
  fp.hq = prob->num_q_heads;
  fp.hkv = prob->num_kv_heads;
  fp.group = prob->num_q_heads / prob->num_kv_heads;
  fp.scale_log2 = prob->softmax_scale * kLog2e;
  fp.accumulate = accumulate;
  PlanBlob blob;
  return with_plan(
      0, prob, q_idx, nq, kv_idx, nkv, ch, may_split, stream, &blob,
      [&](const PlanView& plan) {
        const int64_t slots = may_split ? parts_of(prob, nq, nkv, ch) : 0;
        const ma_status_t room = check_parts(plan.a, fp.hq, slots);
        if (room != MA_OK) return room;
        hipError_t e = hipSuccess;
        if (plan.src) {
          e = launch_plan_copy(wsb, plan.src, plan.bytes, stream);
          if (e != hipSuccess) return hip_fail(e, "work-list copy launch");
        }
        fp.order = order_at(plan.a, plan.src ? wsb : nullptr);
        fp.part_lse = reinterpret_cast<float*>(
            wsb + (plan.src ? align_up(plan.bytes) : 0));
        fp.part_o = fp.part_lse + slots * kFwdBM;
        e = launch_tile_fwd(fp, blob, prob->head_dim, o_f32, stream);
        if (e != hipSuccess) return hip_fail(e, "tile_fwd launch");
        return ok();
      });
}

// Backward of one chunk pair of a tile (the whole tile: one chunk each).
ma_status_t bwd_impl(const ma_problem_t* prob, const int32_t* q_idx,
                     int32_t nq, const int32_t* kv_idx, int32_t nkv,
                     const ma_chunk_t& ch, const void* q, const void* k,
                     const void* v, const void* o, const void* d_o,
                     const float* lse, float* dq, float* dk, float* dv,
                     int32_t accumulate, void* ws, size_t ws_bytes,
                     hipStream_t stream) {
  ma_status_t st = check_tile(prob, q_idx, nq, kv_idx, nkv);
  if (st == MA_OK) st = check_head_dim(prob);
  if (st == MA_OK) st = check_blocks(prob, kBwdBM, kBwdBN);
  if (st == MA_OK) st = check_chunk(prob, ch, kBwdBM, kBwdBN);
  if (st != MA_OK) return st;
  if (accumulate != 0 && accumulate != 1)
    return fail(MA_ERR_INVALID_ARG, "accumulate must be 0 or 1, got %d",
                accumulate);
  const void* ptrs[] = {q, k, v, o, d_o, lse, dq, dk, dv, ws};
  const char* names[] = {"q", "k", "v", "o", "d_o", "lse", "dq", "dk", "dv",
                         "ws"};
  for (int i = 0; i < 10; ++i) {
    if (!ptrs[i]) return fail(MA_ERR_INVALID_ARG, "%s is NULL", names[i]);
    if (!aligned16(ptrs[i]))
      return fail(MA_ERR_INVALID_ARG, "%s is not 16-byte aligned", names[i]);
  }
  const size_t need = bwd_ws_bound(prob, nq, nkv);
  if (ws_bytes < need)
    return fail(MA_ERR_WORKSPACE_TOO_SMALL, "workspace %zu bytes < %zu",
                ws_bytes, need);
  const BwdParts parts = bwd_parts(prob, nq, nkv, ch, false);
  const bool may_split = ws_bytes >= need + parts.bytes;
  char* wsb = static_cast<char*>(ws);
  BwdParams bp{};
  bp.q = static_cast<const uint16_t*>(q);
  bp.k = static_cast<const uint16_t*>(k);
  bp.v = static_cast<const uint16_t*>(v);
  bp.o = static_cast<const uint16_t*>(o);
  bp.d_o = static_cast<const uint16_t*>(d_o);
  bp.lse = lse;
  bp.dq = dq;
  bp.dk = dk;
  bp.dv = dv;
  bp.rows_q = int64_t{nq} * (prob->partition_len / ch.num_q_chunks);
  bp.rows_kv = int64_t{nkv} * (prob->partition_len / ch.num_kv_chunks);
  bp.hq = prob->num_q_heads;
  bp.hkv = prob->num_kv_heads;
  bp.group = prob->num_q_heads / prob->num_kv_heads;
  bp.scale = prob->softmax_scale;
  bp.scale_log2 = prob->softmax_scale * kLog2e;
  bp.accumulate = accumulate;
  PlanBlob blob;
  return with_plan(
      1, prob, q_idx, nq, kv_idx, nkv, ch, may_split, stream, &blob,
      [&](const PlanView& plan) {
        ma_status_t room =
            check_parts(plan.a, bp.hq, may_split ? parts.q : 0);
        if (room == MA_OK)
          room = check_parts(plan.b, bp.hkv, may_split ? parts.kv : 0);
        if (room != MA_OK) return room;
        const size_t row_bytes =
            align_up(static_cast<size_t>(nq) * prob->partition_len *
                     prob->num_q_heads * 4);
        char* at = wsb + align_up(plan.bytes);
        bp.delta = reinterpret_cast<float*>(at);
        bp.lse2 = reinterpret_cast<float*>(at + row_bytes);
        bp.kvparts = reinterpret_cast<float*>(at + 2 * row_bytes);
        bp.qparts =
            reinterpret_cast<float*>(at + 2 * row_bytes + parts.kv_bytes);
        bp.qorder = order_at(plan.a, wsb);
        bp.kvorder = order_at(plan.b, wsb);
        bp.plan_dst = wsb;
        bp.plan_src = plan.src;
        bp.plan_bytes = static_cast<int32_t>(plan.bytes);
        const hipError_t e = launch_tile_bwd(bp, blob, prob->head_dim, stream);
        if (e != hipSuccess) return hip_fail(e, "tile_bwd launch");
        return ok();
      });
}

}  // namespace

extern "C" {

const char* mesh_attn_last_error(void) { return g_last_error.c_str(); }

void mesh_attn_block_shape(int32_t head_dim, int32_t pass, int32_t* bm,
                           int32_t* bn) {
  int32_t m = 0, n = 0;
  if (head_dim == 64 || head_dim == 128) {
    if (pass == 0) {
      m = kFwdBM;
      n = kFwdBN;
    } else if (pass == 1) {
      m = kBwdBM;
      n = kBwdBN;
    }
  }
  if (bm) *bm = m;
  if (bn) *bn = n;
}

ma_status_t mesh_attn_classify(const ma_problem_t* prob, const int32_t* q_idx,
                               int32_t nq, const int32_t* kv_idx, int32_t nkv,
                               int32_t bm, int32_t bn, uint8_t* cls) {
  ma_status_t st = check_tile(prob, q_idx, nq, kv_idx, nkv);
  if (st == MA_OK) st = check_blocks(prob, bm, bn);
  if (st != MA_OK) return st;
  if (!cls) return fail(MA_ERR_INVALID_ARG, "cls is NULL");
  const int64_t P = prob->partition_len;
  const int64_t nqb = nq * P / bm, nkb = nkv * P / bn;
  const int64_t qpb = P / bm, kpb = P / bn;
  for (int64_t qb = 0; qb < nqb; ++qb) {
    const int32_t qp = q_idx[qb / qpb];
    const int64_t q_row = (qb % qpb) * bm;
    const int64_t q_first = token_pos(prob, qp, q_row);
    const int64_t q_last = token_pos(prob, qp, q_row + bm - 1);
    for (int64_t kb = 0; kb < nkb; ++kb) {
      const int32_t kp = kv_idx[kb / kpb];
      const int64_t k_row = (kb % kpb) * bn;
      cls[qb * nkb + kb] = static_cast<uint8_t>(block_class(
          q_first, q_last, token_pos(prob, kp, k_row),
          token_pos(prob, kp, k_row + bn - 1), prob->causal != 0));
    }
  }
  return ok();
}

ma_status_t mesh_attn_worklist(const ma_problem_t* prob, const int32_t* q_idx,
                               int32_t nq, const int32_t* kv_idx, int32_t nkv,
                               int32_t bm, int32_t bn, int32_t* qblk_ptr,
                               ma_run_t* runs, int64_t cap, int64_t* n_runs) {
  ma_status_t st = check_tile(prob, q_idx, nq, kv_idx, nkv);
  if (st == MA_OK) st = check_blocks(prob, bm, bn);
  if (st != MA_OK) return st;
  std::vector<int32_t> ptr;
  std::vector<Run> rl;
  const Slice whole{prob->partition_len, 0};
  build_runs(prob, q_idx, nq, bm, whole, kv_idx, nkv, bn, whole, true, &ptr,
             &rl);
  return export_runs(ptr, rl, qblk_ptr, runs, cap, n_runs);
}

ma_status_t mesh_attn_worklist_kv_major(const ma_problem_t* prob,
                                        const int32_t* q_idx, int32_t nq,
                                        const int32_t* kv_idx, int32_t nkv,
                                        int32_t bm, int32_t bn,
                                        int32_t* kvblk_ptr, ma_run_t* runs,
                                        int64_t cap, int64_t* n_runs) {
  ma_status_t st = check_tile(prob, q_idx, nq, kv_idx, nkv);
  if (st == MA_OK) st = check_blocks(prob, bm, bn);
  if (st != MA_OK) return st;
  std::vector<int32_t> ptr;
  std::vector<Run> rl;
  const Slice whole{prob->partition_len, 0};
  build_runs(prob, kv_idx, nkv, bn, whole, q_idx, nq, bm, whole, false, &ptr,
             &rl);
  return export_runs(ptr, rl, kvblk_ptr, runs, cap, n_runs);
}

size_t mesh_attn_fwd_workspace_size(const ma_problem_t* prob, int32_t nq,
                                    int32_t nkv) {
  if (check_problem(prob) != MA_OK || nq < 1 || nkv < 1) return 0;
  return fwd_ws_bound(prob, nq, nkv) +
         fwd_split_bytes(prob, nq, nkv, kWholeTile, true);
}

size_t mesh_attn_bwd_workspace_size(const ma_problem_t* prob, int32_t nq,
                                    int32_t nkv) {
  if (check_problem(prob) != MA_OK || nq < 1 || nkv < 1) return 0;
  return bwd_ws_bound(prob, nq, nkv) +
         bwd_parts(prob, nq, nkv, kWholeTile, true).bytes;
}

ma_status_t mesh_attn_tile_fwd(const ma_problem_t* prob, const int32_t* q_idx,
                               int32_t nq, const int32_t* kv_idx, int32_t nkv,
                               const void* q, const void* k, const void* v,
                               void* o, ma_dtype_t o_dtype, float* lse,
                               void* ws, size_t ws_bytes, hipStream_t stream) {
  if (o_dtype != MA_BF16 && o_dtype != MA_FP32)
    return fail(MA_ERR_INVALID_ARG, "o_dtype %d invalid", (int)o_dtype);
  return fwd_impl(prob, q_idx, nq, kv_idx, nkv, kWholeTile, q, k, v, o,
                  o_dtype == MA_FP32, lse, 0, ws, ws_bytes, stream);
}

size_t mesh_attn_chunk_fwd_workspace_size(const ma_problem_t* prob,
                                          int32_t nq, int32_t nkv) {
  // A chunk's work list is never longer than the whole tile's.
  return mesh_attn_fwd_workspace_size(prob, nq, nkv);
}

ma_status_t mesh_attn_chunk_fwd(const ma_problem_t* prob, const int32_t* q_idx,
                                int32_t nq, const int32_t* kv_idx, int32_t nkv,
                                const ma_chunk_t* chunk, const void* q,
                                const void* k, const void* v, float* o,
                                float* lse, int32_t accumulate, void* ws,
                                size_t ws_bytes, hipStream_t stream) {
  if (!chunk) return fail(MA_ERR_INVALID_ARG, "chunk is NULL");
  if (accumulate != 0 && accumulate != 1)
    return fail(MA_ERR_INVALID_ARG, "accumulate must be 0 or 1, got %d",
                accumulate);
  return fwd_impl(prob, q_idx, nq, kv_idx, nkv, *chunk, q, k, v, o, true, lse,
                  accumulate, ws, ws_bytes, stream);
}

ma_status_t mesh_attn_tile_fwd_noalloc(const ma_problem_t* prob,
                                       const int32_t* q_idx, int32_t nq,
                                       const int32_t* kv_idx, int32_t nkv,
                                       const void* q, const void* k,
                                       const void* v, void* o,
                                       ma_dtype_t o_dtype, float* lse,
                                       hipStream_t stream) {
  if (o_dtype != MA_BF16 && o_dtype != MA_FP32)
    return fail(MA_ERR_INVALID_ARG, "o_dtype %d invalid", (int)o_dtype);
  ma_status_t st = check_tile(prob, q_idx, nq, kv_idx, nkv);
  if (st == MA_OK) st = check_head_dim(prob);
  if (st == MA_OK) st = check_blocks(prob, kFwdBM, kFwdBN);
  if (st != MA_OK) return st;
  const void* ptrs[] = {q, k, v, o, lse};
  const char* names[] = {"q", "k", "v", "o", "lse"};
  for (int i = 0; i < 5; ++i) {
    if (!ptrs[i]) return fail(MA_ERR_INVALID_ARG, "%s is NULL", names[i]);
    if (!aligned16(ptrs[i]))
      return fail(MA_ERR_INVALID_ARG, "%s is not 16-byte aligned", names[i]);
  }
  if (nq > kNoAllocMaxList || nkv > kNoAllocMaxList)
    return fail(MA_ERR_UNSUPPORTED,
                "noalloc forward: index lists of %d and %d partitions exceed "
                "the maximum of %d", nq, nkv, kNoAllocMaxList);
  const int64_t nqb = int64_t{nq} * prob->partition_len / kFwdBM;
  const size_t need = noalloc_list_bytes(nqb, nkv, prob->num_q_heads);
  if (nqb > kNoAllocMaxQBlocks || need > kNoAllocScratchBytes)
    return fail(MA_ERR_UNSUPPORTED,
                "noalloc forward: the tile (%lld Q blocks, %zu bytes of the "
                "limit's formula) exceeds the scratch maximum (%d Q blocks, "
                "%zu bytes)",
                static_cast<long long>(nqb), need, kNoAllocMaxQBlocks,
                kNoAllocScratchBytes);
  const int64_t items = nqb * prob->num_q_heads;
  if (items > INT32_MAX)
    return fail(MA_ERR_UNSUPPORTED, "noalloc forward: %lld workgroups",
                static_cast<long long>(items));
  void *scratch = nullptr, *parts = nullptr;
  hipError_t e = noalloc_scratch(&scratch, &parts);
  if (e != hipSuccess) return hip_fail(e, "hipGetSymbolAddress(scratch)");
  FwdParams fp{};
  fp.q = static_cast<const uint16_t*>(q);
  fp.k = static_cast<const uint16_t*>(k);
  fp.v = static_cast<const uint16_t*>(v);
  fp.o = o;
  fp.lse = lse;
  fp.rows_q = int64_t{nq} * prob->partition_len;
  fp.hq = prob->num_q_heads;
  fp.hkv = prob->num_kv_heads;
  fp.group = prob->num_q_heads / prob->num_kv_heads;
  fp.scale_log2 = prob->softmax_scale * kLog2e;
  fp.part_lse = static_cast<float*>(parts);
  fp.part_o =
      fp.part_lse + fwd_pass(prob->head_dim).max_parts() * kFwdBM;
  // A short list travels in the kernel's arguments, as with a workspace.
  PlanBlob blob;
  PlanView view;
  plan::Side side[2];
  sides_of(0, prob, q_idx, nq, kv_idx, nkv, kWholeTile, true, side);
  if (inline_plan(side, 1, &blob, &view)) {
    fp.order = order_at(view.a, nullptr);
  } else {
    // The same cut as the call with a workspace of full size.
    NoAllocSplit sp{{}, 0, 0, 0, false};
    if (items <= fwd_pass(prob->head_dim).max_items)
      sp = noalloc_split(prob, q_idx, nq, kv_idx, nkv);
    const bool split = sp.cut.c > 0;
    PassView v;
    v.m = split ? sp.row_pieces : static_cast<int32_t>(nqb);
    v.n_items = v.m * prob->num_q_heads;
    v.n_splits = sp.split_rows;
    v.parts = sp.parts;
    v.is_short = sp.is_short;
    v.mode = split_mode(v.n_items, split, prob->num_kv_heads % kNumXcd == 0,
                        sp.cut.slots);
    v.off_queue = align_up(static_cast<size_t>(v.m) * sizeof(DevRow));
    v.off_splits = v.off_queue + kAlign;
    v.off_runs = v.off_splits + align_up(sp.split_rows * sizeof(DevSplit));
    char* base = static_cast<char*>(scratch);
    fp.order = order_at(v, base);
    PlanBuildParams bp{};
    bp.P = prob->partition_len;
    bp.n = prob->num_partitions;
    bp.layout = prob->layout;
    bp.causal = prob->causal;
    bp.nq = nq;
    bp.nkv = nkv;
    bp.bm = kFwdBM;
    bp.bn = kFwdBN;
    bp.nqb = static_cast<int32_t>(nqb);
    bp.nkbp = prob->partition_len / kFwdBN;
    bp.cut = sp.cut;
    bp.m = v.m;
    bp.mode = v.mode;
    bp.rows = reinterpret_cast<DevRow*>(base + v.off_rows);
    bp.runs = reinterpret_cast<DevRun*>(base + v.off_runs);
    bp.splits = reinterpret_cast<DevSplit*>(base + v.off_splits);
    bp.queue = reinterpret_cast<int32_t*>(base + v.off_queue);
    for (int32_t i = 0; i < nq; ++i) bp.q_idx[i] = q_idx[i];
    for (int32_t i = 0; i < nkv; ++i) bp.kv_idx[i] = kv_idx[i];
    e = launch_fwd_plan_build(bp, stream);
    if (e != hipSuccess) return hip_fail(e, "noalloc work-list build launch");
  }
  e = launch_tile_fwd(fp, blob, prob->head_dim, o_dtype == MA_FP32, stream);
  if (e != hipSuccess) return hip_fail(e, "tile_fwd launch");
  return ok();
}

ma_status_t mesh_attn_lse_merge(int32_t k_parts, int64_t rows, int32_t heads,
                                int32_t head_dim, const void* o_parts,
                                ma_dtype_t in_dtype, const float* lse_parts,
                                void* o_out, ma_dtype_t out_dtype,
                                float* lse_out, hipStream_t stream) {
  if (k_parts < 1 || k_parts > 4096)
    return fail(MA_ERR_INVALID_ARG, "k_parts %d outside [1, 4096]", k_parts);
  if (rows < 0) return fail(MA_ERR_INVALID_ARG, "rows %lld < 0", (long long)rows);
  if (heads < 1) return fail(MA_ERR_INVALID_ARG, "heads %d < 1", heads);
  if (head_dim < 8 || head_dim > 256 || head_dim % 8 != 0)
    return fail(MA_ERR_UNSUPPORTED, "head_dim %d: need a multiple of 8 in "
                "[8, 256]", head_dim);
  if ((in_dtype != MA_BF16 && in_dtype != MA_FP32) ||
      (out_dtype != MA_BF16 && out_dtype != MA_FP32))
    return fail(MA_ERR_INVALID_ARG, "dtype invalid (in %d, out %d)",
                (int)in_dtype, (int)out_dtype);
  if (rows == 0) return ok();
  const void* ptrs[] = {o_parts, lse_parts, o_out, lse_out};
  const char* names[] = {"o_parts", "lse_parts", "o_out", "lse_out"};
  for (int i = 0; i < 4; ++i) {
    if (!ptrs[i]) return fail(MA_ERR_INVALID_ARG, "%s is NULL", names[i]);
    if (!aligned16(ptrs[i]))
      return fail(MA_ERR_INVALID_ARG, "%s is not 16-byte aligned", names[i]);
  }
  if (rows * heads > (int64_t{1} << 40))
    return fail(MA_ERR_INVALID_ARG, "rows * heads too large");
  MergeParams mp{o_parts, lse_parts, o_out, lse_out, rows, k_parts, heads,
                 head_dim};
  hipError_t e = launch_lse_merge(mp, in_dtype == MA_FP32,
                                  out_dtype == MA_FP32, stream);
  if (e != hipSuccess) return hip_fail(e, "lse_merge launch");
  return ok();
}

ma_status_t mesh_attn_tile_bwd(const ma_problem_t* prob, const int32_t* q_idx,
                               int32_t nq, const int32_t* kv_idx, int32_t nkv,
                               const void* q, const void* k, const void* v,
                               const void* o, const void* d_o,
                               const float* lse, float* dq, float* dk,
                               float* dv, int32_t accumulate, void* ws,
                               size_t ws_bytes, hipStream_t stream) {
  return bwd_impl(prob, q_idx, nq, kv_idx, nkv, kWholeTile, q, k, v, o, d_o,
                  lse, dq, dk, dv, accumulate, ws, ws_bytes, stream);
}

size_t mesh_attn_chunk_bwd_workspace_size(const ma_problem_t* prob,
                                          int32_t nq, int32_t nkv) {
  // A chunk's work lists and row buffers never exceed the whole tile's.
  return mesh_attn_bwd_workspace_size(prob, nq, nkv);
}

ma_status_t mesh_attn_chunk_bwd(const ma_problem_t* prob, const int32_t* q_idx,
                                int32_t nq, const int32_t* kv_idx, int32_t nkv,
                                const ma_chunk_t* chunk, const void* q,
                                const void* k, const void* v, const void* o,
                                const void* d_o, const float* lse, float* dq,
                                float* dk, float* dv, int32_t accumulate,
                                void* ws, size_t ws_bytes, hipStream_t stream) {
  if (!chunk) return fail(MA_ERR_INVALID_ARG, "chunk is NULL");
  return bwd_impl(prob, q_idx, nq, kv_idx, nkv, *chunk, q, k, v, o, d_o, lse,
                  dq, dk, dv, accumulate, ws, ws_bytes, stream);
}

}  // extern "C"
