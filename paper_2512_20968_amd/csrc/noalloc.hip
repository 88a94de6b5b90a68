// The allocation-free forward of tiles whose work list does not fit a kernel
// argument: the list is built on the device, into a fixed scratch array that
// every call on a GPU shares, instead of being built on the host and copied
// from pinned memory into a caller-provided workspace.  Everything a launch
// needs travels in kernel arguments (the index lists included), so the call
// allocates nothing, host or device, and never waits.
//
// The builder reproduces the host's list (plan.h): the Section 3.7 rule per
// block pair, runs in KV-list order, and the order table, with one workgroup
// of 1024 threads.  Along one KV partition a Q block's classes only fall
// (positions grow with the row under both layouts), so each (Q block, KV
// partition) pair has a FULL prefix and a PARTIAL middle whose lengths are
// found by binary search.

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>

#include "internal.h"
#include "mesh_attn.h"

namespace mesh_attn {
namespace {

// The scratch arrays of the allocation-free forward, on every GPU the library
// runs on, held until the process ends: the lists, and the partial results.  Host code
// must never pass its name to a kernel (the name is a host-side stand-in):
// noalloc_scratch() gives the device address.
__device__ __align__(256) char scratch[kNoAllocScratchBytes +
                                       kNoAllocTableBytes];
__device__ __align__(256) char part_scratch[kNoAllocPartBytes];

constexpr int kBuildThreads = 1024;

__device__ int64_t tok_pos(const PlanBuildParams& p, int part, int64_t row) {
  return p.layout == 1 ? row * p.n + part : int64_t{part} * p.P + row;
}

// Length of the prefix of [0, p.nkbp) on which `pred` holds (pred holds on a
// prefix).
template <class F>
__device__ int prefix_len(int nkbp, F pred) {
  int lo = 0, hi = nkbp;  // pred(lo - 1) holds, pred(hi) fails
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (pred(mid))
      lo = mid + 1;
    else
      hi = mid;
  }
  return lo;
}

struct PairRuns {
  int nfull, nvis;        // FULL blocks [0, nfull), PARTIAL [nfull, nvis)
  int32_t qp, kp;
  int64_t q_row0;
};

__device__ PairRuns pair_runs(const PlanBuildParams& p, int qb, int b) {
  const int qpb = p.P / p.bm;
  PairRuns r;
  r.qp = p.q_idx[qb / qpb];
  r.kp = p.kv_idx[b];
  r.q_row0 = int64_t{qb % qpb} * p.bm;
  if (!p.causal) {
    r.nfull = r.nvis = p.nkbp;
    return r;
  }
  const int64_t qf = tok_pos(p, r.qp, r.q_row0);
  const int64_t ql = tok_pos(p, r.qp, r.q_row0 + p.bm - 1);
  const int kp = r.kp;
  // FULL: every key of the block at or before every query of the Q block.
  r.nfull = prefix_len(p.nkbp, [&](int kb) {
    return tok_pos(p, kp, int64_t{kb} * p.bn + p.bn - 1) <= qf;
  });
  // Not EMPTY: some key of the block at or before some query.
  r.nvis = prefix_len(p.nkbp, [&](int kb) {
    return tok_pos(p, kp, int64_t{kb} * p.bn) <= ql;
  });
  return r;
}

// Mask offset of a run starting at KV block kb0 (see DevRun).
__device__ int32_t run_delta(const PlanBuildParams& p, const PairRuns& r,
                             int kb0) {
  const int64_t k_row0 = int64_t{kb0} * p.bn;
  if (p.layout == 1)
    return static_cast<int32_t>((r.q_row0 - k_row0) + (r.qp >= r.kp ? 0 : -1));
  return static_cast<int32_t>(tok_pos(p, r.qp, r.q_row0) -
                              tok_pos(p, r.kp, k_row0));
}

// The runs of Q block qb, FULL runs that continue each other in the KV buffer
// as one; emit(run) for each.  Returns the blocks.
template <class F>
__device__ int row_runs(const PlanBuildParams& p, int qb, F emit) {
  int work = 0;
  DevRun full{0, 0, MA_CLS_FULL, 0};  // the FULL run being extended
  for (int b = 0; b < p.nkv; ++b) {
    const PairRuns r = pair_runs(p, qb, b);
    work += r.nvis;
    if (r.nfull > 0) {
      const int blk0 = b * p.nkbp;
      if (full.nblk > 0 && full.blk0 + full.nblk == blk0) {
        full.nblk += r.nfull;
      } else {
        if (full.nblk > 0) emit(full);
        full = DevRun{blk0, r.nfull, MA_CLS_FULL, run_delta(p, r, 0)};
      }
    }
    if (r.nvis > r.nfull) {
      if (full.nblk > 0) emit(full);
      full.nblk = 0;
      emit(DevRun{b * p.nkbp + r.nfull, r.nvis - r.nfull, MA_CLS_PARTIAL,
                  run_delta(p, r, r.nfull)});
    }
  }
  if (full.nblk > 0) emit(full);
  return work;
}

// Exclusive scan of one value per thread of the workgroup, and the total: in
// each wave, then over the waves' sums.
__device__ int scan_before(int* s_wave, int v, int* total) {
  constexpr int kWaves = kBuildThreads / 64;
  const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
  int x = v;
  for (int off = 1; off < 64; off <<= 1) {
    const int y = __shfl_up(x, off);
    if (lane >= off) x += y;
  }
  __syncthreads();  // the reads of a scan before this one
  if (lane == 63) s_wave[wave] = x;
  __syncthreads();
  int base = 0, sum = 0;
#pragma unroll
  for (int i = 0; i < kWaves; ++i) {
    base += i < wave ? s_wave[i] : 0;
    sum += s_wave[i];
  }
  *total = sum;
  return base + x - v;
}

__global__ __launch_bounds__(kBuildThreads) void fwd_plan_build_kernel(
    PlanBuildParams p) {
  __shared__ int s_work[kNoAllocMaxQBlocks];
  __shared__ int s_run[kNoAllocMaxQBlocks];     // first run of each Q block
  // Split tiles: blocks, Q block and index of each piece (before ranking), first
  // piece and first partial (or -1) of each Q block.  Whole items: piece i is Q
  // block i.  The indexes lie behind the work of the (at most kSplitMaxRows) Q
  // blocks of a split tile.
  __shared__ int s_len[kSplitMaxPieces];
  __shared__ uint16_t s_row[kSplitMaxPieces];
  __shared__ uint16_t s_pre[kSplitMaxRows];
  __shared__ int16_t s_part[kSplitMaxRows];
  __shared__ int s_wave[kBuildThreads / 64];
  uint16_t* s_idx = reinterpret_cast<uint16_t*>(s_work + kSplitMaxRows);
  static_assert(kSplitMaxPieces * 2 <=
                    (kNoAllocMaxQBlocks - kSplitMaxRows) * 4,
                "room for the piece indexes");
  const int t = threadIdx.x;
  const bool cut = p.cut.c > 0;
  // Thread t owns a contiguous segment of Q blocks for the run list.
  const int seg = (p.nqb + kBuildThreads - 1) / kBuildThreads;
  const int lo = min(t * seg, p.nqb);
  const int hi = min(lo + seg, p.nqb);
  int cnt = 0;
  for (int qb = lo; qb < hi; ++qb)
    s_work[qb] = row_runs(p, qb, [&](const DevRun&) { ++cnt; });
  int n_runs = 0;
  int at = scan_before(s_wave, cnt, &n_runs);
  for (int qb = lo; qb < hi; ++qb) {
    s_run[qb] = at;
    row_runs(p, qb, [&](const DevRun& r) { p.runs[at++] = r; });
  }
  if (cut) {
    // Pieces and split rows of the Q blocks before each, in one scan (at most
    // kSplitMaxPieces and kSplitMaxRows); the partials follow, as a row that is
    // not split is one piece and no partial.
    constexpr int kBits = 12;
    static_assert(kSplitMaxPieces < 1 << kBits && kSplitMaxRows < 1 << kBits,
                  "two counts in one value");
    int sum = 0;
    for (int qb = lo; qb < hi; ++qb) {
      const int n = split::num_pieces(p.cut, qb, s_work[qb]);
      sum += n + ((n > 1) << kBits);
    }
    int all = 0;
    int before = scan_before(s_wave, sum, &all);
    for (int qb = lo; qb < hi; ++qb) {
      const int w = s_work[qb], n = split::num_pieces(p.cut, qb, w);
      const int pre = before & ((1 << kBits) - 1), splits = before >> kBits;
      const int part = pre - (qb - splits);
      s_pre[qb] = static_cast<uint16_t>(pre);
      s_part[qb] = static_cast<int16_t>(n > 1 ? part : -1);
      if (n > 1) p.splits[splits] = DevSplit{qb, part, n};
      int begin = 0;
      for (int j = 0; j < n; ++j) {
        const int end = split::piece_begin(w, n, j + 1);
        s_row[pre + j] = static_cast<uint16_t>(qb);
        s_idx[pre + j] = static_cast<uint16_t>(j);
        s_len[pre + j] = end - begin;
        begin = end;
      }
      before += n + ((n > 1) << kBits);
    }
  }
  __syncthreads();  // and the runs, read back below
  // Ranks: longest first, or in one round by piece index; ties in table order.
  const int* len_of = cut ? s_len : s_work;
  const bool by_len = p.mode != kModeOneRound;
  for (int i = t; i < p.m; i += kBuildThreads) {
    const int qb = cut ? s_row[i] : i, idx = cut ? s_idx[i] : 0;
    const int len = len_of[i];
    int before = 0, same = 0, same_before = 0;
    auto count = [&](auto key) {
      const int k = key(i);
#pragma unroll 8
      for (int i2 = 0; i2 < p.m; ++i2) {
        const int k2 = key(i2);
        before += k2 < k;
        same += k2 == k;
        same_before += (k2 == k) & (i2 < i);
      }
    };
    if (by_len)
      count([&](int x) { return -len_of[x]; });
    else
      count([&](int x) { return int{s_idx[x]}; });
    const int run_b = s_run[qb], run_e = qb + 1 < p.nqb ? s_run[qb + 1] : n_runs;
    int run = run_b, off = 0;
    if (idx > 0) {
      const int w = s_work[qb];
      off = split::piece_begin(w, split::num_pieces(p.cut, qb, w), idx);
      while (off >= p.runs[run].nblk) off -= p.runs[run++].nblk;
    }
    const int part = cut && s_part[qb] >= 0 ? s_part[qb] + idx : -1;
    p.rows[before + same_before] = DevRow{qb,   run, off,   len,   part,
                                          0,    run_b, run_e, before, same};
  }
  if (t < kNumXcd) p.queue[t] = 0;
}

// Device address of the scratch array, per device (each GPU holds its own
// copy at its own address).
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};
void* g_parts_ptr[kMaxDevices] = {};

}  // namespace

hipError_t noalloc_scratch(void** ptr, void** parts) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_ptr[dev] == nullptr) {
    // Once per device, with that device current.
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (p == nullptr) return hipErrorInvalidSymbol;
    void* q = nullptr;
    e = hipGetSymbolAddress(&q, HIP_SYMBOL(part_scratch));
    if (e != hipSuccess) return e;
    if (q == nullptr) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = p;
    g_parts_ptr[dev] = q;
  }
  *ptr = g_scratch_ptr[dev];
  *parts = g_parts_ptr[dev];
  return hipSuccess;
}

hipError_t launch_fwd_plan_build(const PlanBuildParams& p,
                                 hipStream_t stream) {
  hipLaunchKernelGGL(fwd_plan_build_kernel, dim3(1), dim3(kBuildThreads), 0,
                     stream, p);
  return hipGetLastError();
}

}  // namespace mesh_attn
