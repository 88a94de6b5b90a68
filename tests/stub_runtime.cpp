// A stand-in for the GPU under the library's host code, for CPU tests: linked
// with csrc/host.cpp instead of the HIP runtime and the kernels.  The work of a
// stream (copies of work lists, events) runs only when the test says so, so
// that the lifetime of the pinned work lists can be checked; a launch checks
// that everything its kernels write in the workspace lies inside it.

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <map>
#include <mutex>
#include <vector>

#include "internal.h"

using namespace mesh_attn;

namespace {

std::recursive_mutex mu;

struct Event {
  long recorded = 0, done = 0;
};
struct Op {
  Event* ev = nullptr;  // an event, or a copy:
  char* dst = nullptr;
  const char* src = nullptr;
  std::vector<char> want;  // the source when the copy was enqueued
};

std::map<hipStream_t, std::deque<Op>> ops;
char *ws = nullptr, *ws_end = nullptr;
int32_t out_of_range = 0, stale = 0, pinned = 0, launches = 0;
int32_t fail_launch = 0, fail_event = 0;
int32_t last[2][7];
void (*hook)() = nullptr;

void enqueue_copy(void* dst, const void* src, size_t bytes,
                  hipStream_t stream) {
  Op o;
  o.dst = static_cast<char*>(dst);
  o.src = static_cast<const char*>(src);
  o.want.assign(o.src, o.src + bytes);
  if (o.dst < ws || o.dst + bytes > ws_end) ++out_of_range;
  ops[stream].push_back(std::move(o));
}

void inside(const void* at, size_t bytes, const void* end) {
  const char* p = static_cast<const char*>(at);
  if (p < ws || p + bytes > static_cast<const char*>(end)) ++out_of_range;
}

void note(int i, const DevOrder& o) {
  const int32_t v[7] = {o.inline_list, o.m, o.n_items, o.mode,
                        o.parts,       o.n_splits, o.is_short};
  std::memcpy(last[i], v, sizeof v);
}

hipError_t launched() {
  ++launches;
  if (fail_launch > 0) {
    --fail_launch;
    return hipErrorLaunchFailure;
  }
  return hipSuccess;
}

}  // namespace

extern "C" {

const char* hipGetErrorString(hipError_t) { return "stub error"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t bytes, unsigned) {
  std::lock_guard<std::recursive_mutex> lock(mu);
  ++pinned;
  *p = std::malloc(bytes);
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  *e = reinterpret_cast<hipEvent_t>(new Event);
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t stream) {
  std::lock_guard<std::recursive_mutex> lock(mu);
  if (fail_event > 0) {
    --fail_event;
    return hipErrorInvalidHandle;
  }
  Op o;
  o.ev = reinterpret_cast<Event*>(e);
  ++o.ev->recorded;
  ops[stream].push_back(std::move(o));
  return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e) {
  std::lock_guard<std::recursive_mutex> lock(mu);
  const Event* ev = reinterpret_cast<Event*>(e);
  return ev->done == ev->recorded ? hipSuccess : hipErrorNotReady;
}

void stub_workspace(char* p, size_t bytes) {
  ws = p;
  ws_end = p + bytes;
}
// Runs the pending operations of the stream.
void stub_run(hipStream_t stream) {
  std::lock_guard<std::recursive_mutex> lock(mu);
  for (; !ops[stream].empty(); ops[stream].pop_front()) {
    Op& o = ops[stream].front();
    if (o.ev) {
      ++o.ev->done;
    } else {
      if (std::memcmp(o.src, o.want.data(), o.want.size()) != 0) ++stale;
      std::memcpy(o.dst, o.src, o.want.size());
    }
  }
}
void stub_fail(int32_t n_launches, int32_t n_events) {
  fail_launch = n_launches;
  fail_event = n_events;
}
// Called once, inside the next launch.
void stub_hook(void (*f)()) { hook = f; }
// {accesses outside the workspace, copies whose source changed before they
// ran, pinned buffers allocated, launches}
void stub_counts(int32_t out[4]) {
  const int32_t v[4] = {out_of_range, stale, pinned, launches};
  std::memcpy(out, v, sizeof v);
}
// {list in the arguments, entries, items, mode, partials per head, split rows,
// short items} of the last launch's order(s): the forward's, or dQ's and
// dK/dV's.
void stub_last(int32_t out[2][7]) { std::memcpy(out, last, sizeof last); }

}  // extern "C"

namespace mesh_attn {

hipError_t launch_plan_copy(void* dst, const void* src, size_t bytes,
                            hipStream_t stream) {
  std::lock_guard<std::recursive_mutex> lock(mu);
  enqueue_copy(dst, src, bytes, stream);
  return hipSuccess;
}

hipError_t launch_tile_fwd(const FwdParams& p, const PlanBlob&, int head_dim,
                           bool, hipStream_t) {
  if (void (*f)() = hook) {
    hook = nullptr;
    f();
  }
  std::lock_guard<std::recursive_mutex> lock(mu);
  note(0, p.order);
  const size_t parts = size_t{1} * p.order.parts * p.hq;
  const DevSplit* splits_end = p.order.splits + p.order.n_splits;
  if (!p.order.inline_list && p.order.runs >= (const void*)p.order.splits &&
      p.order.runs < (const void*)splits_end)
    ++out_of_range;
  if (parts > 0) {
    inside(p.part_lse, parts * kFwdBM * 4, p.part_o);
    inside(p.part_o, parts * kFwdBM * head_dim * 4, ws_end);
  }
  return launched();
}

hipError_t launch_tile_bwd(const BwdParams& p, const PlanBlob&, int head_dim,
                           hipStream_t stream) {
  std::lock_guard<std::recursive_mutex> lock(mu);
  note(0, p.qorder);
  note(1, p.kvorder);
  if (p.plan_src)
    enqueue_copy(p.plan_dst, p.plan_src, p.plan_bytes, stream);
  inside(p.plan_dst, p.plan_bytes, p.delta);
  inside(p.delta, p.rows_q * p.hq * 4, p.lse2);
  const size_t tile = size_t{128} * head_dim * 4;
  const size_t kv = size_t{1} * p.kvorder.parts * p.hkv;
  const size_t q = size_t{1} * p.qorder.parts * p.hq;
  inside(p.lse2, p.rows_q * p.hq * 4, p.kvparts);
  if (kv > 0) inside(p.kvparts, kv * 2 * tile, p.qparts);
  if (q > 0) inside(p.qparts, q * tile, ws_end);
  return launched();
}

hipError_t launch_lse_merge(const MergeParams&, bool, bool, hipStream_t) {
  return launched();
}

namespace {
std::vector<char> lists(kNoAllocScratchBytes + kNoAllocTableBytes);
}

hipError_t noalloc_scratch(void** ptr, void** parts) {
  static std::vector<char> partials(kNoAllocPartBytes);
  *ptr = lists.data();
  *parts = partials.data();
  stub_workspace(partials.data(), partials.size());
  return hipSuccess;
}

// The lists in order, none into the next, the runs (at most two per Q block and
// KV partition) up to the array's end.
hipError_t launch_fwd_plan_build(const PlanBuildParams& p, hipStream_t) {
  const void* at[] = {p.rows, p.queue, p.splits, p.runs};
  const size_t bytes[] = {p.m * sizeof(DevRow), kNumXcd * 4,
                          0,  // their number: launch_tile_fwd
                          size_t{2} * p.nqb * p.nkv * sizeof(DevRun)};
  const char* end = lists.data();
  for (int i = 0; i < 4; ++i) {
    const char* begin = static_cast<const char*>(at[i]);
    if (begin < end) ++out_of_range;
    end = begin + bytes[i];
  }
  if (end > lists.data() + lists.size()) ++out_of_range;
  return launched();
}

}  // namespace mesh_attn
