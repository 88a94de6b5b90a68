// Internal interface between the host library (host.cpp) and the HIP kernel
// translation units.  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

#include "split.h"

namespace mesh_attn {

// Forward block shape: 8 waves x 32 query rows, 64 keys per LDS stage.
constexpr int kFwdBM = 256;
constexpr int kFwdBN = 64;

// Backward block shapes.
constexpr int kBwdBM = 128;  // Q rows per dQ workgroup (4 waves x 32)
constexpr int kBwdBN = 128;  // KV rows per dK/dV workgroup (4 waves x 32)

// One run of consecutive KV blocks of one KV list entry, as the kernels read
// it: x = first KV block (index into the tile's KV buffer, in blocks of the
// pass's KV block size), y = number of blocks, z = class (MA_CLS_*),
// w = position of the Q block's first row minus position of the run's first
// key (the causal mask of a PARTIAL run: key j of the run is hidden from
// query i of the block iff j - i > w).
struct DevRun {
  int32_t blk0, nblk, cls, delta;
};

// Entry of a pass's order table: the workgroup's share of an item, nblk blocks
// of block row `row` from block `off` of run `run` on (the dK/dV items walk
// their runs [run_b, run_e) once per query head of the group; the share
// starts in walk `walk`).  part >= 0: it is a piece of a split item and leaves
// its partial result in slot head * parts + part.  The entry's rank class is
// [before, before + same) (split.h).
struct DevRow {
  int32_t row, run, off, nblk, part, walk, run_b, run_e, before, same;
};

// A row whose items are split: the partial results of head h are slots
// [h * parts + part, .. + nparts).
struct DevSplit {
  int32_t row, part, nparts;
};

// The order of a pass as its kernels get it.
struct DevOrder {
  const DevRow* rows;  // [m]
  const DevRun* runs;
  const DevSplit* splits;  // [n_splits]
  int32_t* queue;      // [8] items taken from each XCD lane, 0 at launch; used
                       // from kQueuedMinItems items on
  int32_t m, n_items;  // table entries; times the heads: workgroup items
  int32_t mode, parts, n_splits;
  int32_t is_short;     // the forward's waves split the keys (fwd_is_short)
  int32_t inline_list;  // the three lists are in the PlanBlob argument
  int32_t off_runs, off_splits;  // at these offsets (rows first)
};

// A small work list travels in the kernel's arguments instead of the
// workspace: no upload, and no pinned copy to keep until one is done.  Kernel
// arguments stay within 4 KB; 512 bytes are left for the other ones.  A list
// that has to be copied costs a copy kernel and an event: 64 items of 1024
// blocks (16 rows in 4 pieces each, 3.1 KB) 483 us a call with the copy, 475
// in the arguments; calls with shorter lists the same within 0.6 % when the
// arguments grow from 3 KB.
constexpr int kInlinePlan = 3584;
struct PlanBlob {
  alignas(16) char bytes[kInlinePlan];
};

struct FwdParams {
  const uint16_t* q;   // bf16 [rows_q][hq][d]
  const uint16_t* k;   // bf16 [rows_kv][hkv][d]
  const uint16_t* v;
  void* o;             // bf16 or f32 [rows_q][hq][d]
  float* lse;          // [hq][rows_q]
  DevOrder order;
  int64_t rows_q;
  int32_t hq, hkv, group;
  float scale_log2;    // softmax scale * log2(e)
  int32_t accumulate;  // 1: fold into the float32 (O, LSE) already stored
  // Partial results of split items, [part][kFwdBM][d] and [part][kFwdBM] (log2
  // units).
  float* part_o;
  float* part_lse;
};

// The forward as the cut of long items sees it.  d = 128: one workgroup per
// compute unit (its eight waves of 256 registers fill the SIMDs); items of 4
// and 64 KV blocks measured 14.3 and 100.8 us (1.44 us per block and six
// blocks of overhead); folding 256 partials of 256 x 128 takes 7-9 us, and
// writing them about as long.  d = 64: two workgroups per compute unit, 2.37 us
// per block each; a whole item with a compute unit to itself takes 46, 80 and
// 152 us for 32, 64 and 128 blocks, half of that rate, while a cut in two then
// fills the unit and gains nothing.  Its price is set a little above (the
// estimates of cuts are, too), where it tells the cuts that measured slower from
// those that measured faster, microseconds whole / cut:
//   192 items of  32 blocks  45.8/52.7 (whole)   112 of  32  43.3/35.2 (cut)
//   192 of        64         79.9/89.6 (whole)   168 of  64  79.7/68.0 (cut)
//   256 of        64         89.1/96.4 (whole)   128 of  64  79.8/55.1 (cut)
//   192 of       128        151.8/156  (whole)   256 of 256   325/313  (cut)
constexpr split::Pass kFwdPass128{256, 2048, 6, 4, 2, 20};
constexpr split::Pass kFwdPass64{512, 2048, 4, 4, 2, 60, 57, 7};
constexpr const split::Pass& fwd_pass(int head_dim) {
  return head_dim == 128 ? kFwdPass128 : kFwdPass64;
}

// Workgroup items of the forward and of both backward kernels.  The XCDs of
// the part run at different speeds (a few per cent apart under load) while
// the dispatcher gives each an eighth of the workgroups, so on launches with
// many items per compute unit the last quarter of every XCD lane of the item
// order is taken from per-lane counters: the first queued_static_slots(n)
// workgroups take slot blockIdx.x, the others the next remaining item of
// their XCD's lane or else of another lane, and about one in eight more of
// them are launched than remaining items, so an XCD that runs faster takes
// more of the last items.  Below kQueuedMinItems (16 items per compute unit
// of the 256-CU part) every slot is static and no counter is read.
constexpr int64_t kQueuedMinItems = 4096;
__host__ __device__ inline int64_t queued_static_slots(int64_t n_items) {
  return n_items >= kQueuedMinItems ? (n_items / 8) * 3 / 4 * 8 : n_items;
}
__host__ __device__ inline int64_t queued_launch_grid(int64_t n_items) {
  const int64_t fixed = queued_static_slots(n_items);
  const int64_t dyn = n_items - fixed;
  return dyn > 0 ? fixed + (dyn + dyn / 8 + 8 + 7) / 8 * 8 : fixed;
}

// The tile kernel and, if items are split, the fold of their partial results.
hipError_t launch_tile_fwd(const FwdParams& p, const PlanBlob& blob,
                           int head_dim, bool out_f32, hipStream_t stream);

// Copies `bytes` (a multiple of 16) of a work list from pinned host memory to
// the device, by a kernel.  hipMemcpyAsync on the same stream held the next
// kernel back by 18 to 26 us where it went through a copy engine (lists above
// some 10 KB) and by 5 to 10 us below; this takes 3 to 5 us.
hipError_t launch_plan_copy(void* dst, const void* src, size_t bytes,
                            hipStream_t stream);

// Whether the forward of a tile of `items` items, the longest of `longest` KV
// blocks, runs with the keys split over the waves of 32-row workgroups: its
// 8 * items workgroups (128 KB of LDS each) fit the 256 compute units in one or
// two rounds, and its waves, which wait for the loads of every block, get few
// enough of them.  Microseconds a call, this / 256-row workgroups with long
// items split:
//   d = 64   8 blocks   16         32         64         128
//   4 items  8.5/15     7.9/18     9.7/14.5   15.9/17.3  30.9/21.1
//   32       7.8/15     7.8/22     12.6/22.3  21.5/31.4  37.5/40.0
//   64       9.9/15.1   12.7/21.9  21.7/26.6  37.7/38.6  78/56
//   128      18.5/15.6  23.7/26.9  41.6/37.7
//   d = 128  8          16         32         64
//   4        7.9/20     11.5/18.3  19.2/19.3  35.9/23.3
//   32       8.6/20     13.4/26.5  22.2/31.8  37.8/36.2
//   64       15.2/20.1  25.0/31.1  41.2/38.6
constexpr bool fwd_is_short(int64_t items, int32_t longest, int head_dim) {
  return items <= 64 &&
         longest * (items > 32 ? 2 : 1) <= (head_dim == 64 ? 64 : 32);
}

struct MergeParams {
  const void* o_parts;
  const float* lse_parts;
  void* o_out;
  float* lse_out;
  int64_t rows;
  int32_t k_parts, heads, head_dim;
};

hipError_t launch_lse_merge(const MergeParams& p, bool in_f32, bool out_f32,
                            hipStream_t stream);

struct BwdParams {
  const uint16_t* q;
  const uint16_t* k;
  const uint16_t* v;
  const uint16_t* o;
  const uint16_t* d_o;
  const float* lse;
  float* dq;
  float* dk;
  float* dv;
  float* delta;        // workspace [hq][rows_q]: rowsum(dO * O)
  float* lse2;         // workspace [hq][rows_q]: LSE * log2(e), -inf -> +inf
  // dQ: Q blocks of kBwdBM rows walk KV blocks of kBwdBN.  dK/dV: KV blocks
  // walk Q blocks, once per query head of the group; a run's delta is q-first
  // minus kv-first in both.  Both lists are in the workspace once the prep
  // kernel has run, which copies them there: plan_bytes (a multiple of 16) from
  // plan_src (pinned host memory; null: the PlanBlob argument) to plan_dst.
  DevOrder qorder, kvorder;
  void* plan_dst;
  const void* plan_src;
  int32_t plan_bytes;
  int64_t rows_q, rows_kv;
  int32_t hq, hkv, group;
  float scale, scale_log2;
  int32_t accumulate;
  // Partial results of split items, [part][dV, dK][kBwdBN][d] and
  // [part][kBwdBM][d].
  float* kvparts;
  float* qparts;
};
static_assert(sizeof(FwdParams) + sizeof(PlanBlob) <= 4096 &&
                  sizeof(BwdParams) + sizeof(PlanBlob) <= 4096,
              "kernel arguments");

// The backward passes as the cut of long items sees them; a block is 128 x 128.
// The two passes share a launch.  d = 128: two workgroups of either per compute
// unit, dK/dV first.  The numbers are fitted to whole launches, not the
// residency: cuts for 256 places of dK/dV and 512 of dQ were as good as or better
// than 512/512, 384/384 and 512/256 on a grid of 187 tiles (geometric mean 2 to
// 4 % slower with those).  But dQ items that are left whole for 512 places (they
// fill one round, or nearly whole rounds) have only one place per compute unit
// beside a dK/dV item: looked at again for 256 places, the 14 tiles of the grid
// that are then cut take 5 to 19 % less, microseconds before / now:
//   256 dK/dV items of 384 blocks, 384 dQ of 256   2630/2323 (2526 as launches
//   256 of  48, 384 of  32                          347/316   (343) of their own)
//   512 of 672, 1344 of 256                        8865/8159  (8552)
// d = 64: three workgroups of either per compute unit, 6.1 and 4.6 us per block
// each; each pass gets half of the 768 places (fitted on one 4K-token tile of 12
// heads: 66 us so, 72 with 768 places each, 78 with 512 and 256).
constexpr split::Pass kDkdvPass128{256, 2048, 3, 2, 1, 40};
constexpr split::Pass kDkdvPass64{384, 2048, 2, 2, 1, 100};
constexpr split::Pass kDqBesideDkdv128{256, 4096, 2, 4, 2, 60};
constexpr split::Pass kDqPass128{512, 4096, 2, 2, 1, 120, 0, 0,
                                 &kDqBesideDkdv128};
constexpr split::Pass kDqPass64{384, 4096, 2, 2, 1, 200};
constexpr const split::Pass& dkdv_pass(int head_dim) {
  return head_dim == 128 ? kDkdvPass128 : kDkdvPass64;
}
constexpr const split::Pass& dq_pass(int head_dim) {
  return head_dim == 128 ? kDqPass128 : kDqPass64;
}

hipError_t launch_tile_bwd(const BwdParams& p, const PlanBlob& blob,
                           int head_dim, hipStream_t stream);

// ---------------------------------------------------------------------------
// Allocation-free forward (noalloc.hip): the work list is built on the device
// into a fixed scratch array instead of a caller workspace.
// ---------------------------------------------------------------------------

constexpr size_t kNoAllocScratchBytes = size_t{8} << 20;  // per GPU
constexpr int kNoAllocMaxList = 256;      // partitions per index list
constexpr int kNoAllocMaxQBlocks = 4096;  // forward Q blocks of the tile

// Partial results of a split tile: the most slots there are.
constexpr size_t part_bytes(const split::Pass& ps, int head_dim) {
  return size_t{1} * ps.max_parts() * kFwdBM * (head_dim + 1) * 4;
}
constexpr size_t kNoAllocPartBytes =
    part_bytes(kFwdPass128, 128) > part_bytes(kFwdPass64, 64)
        ? part_bytes(kFwdPass128, 128)
        : part_bytes(kFwdPass64, 64);
// Block rows of a tile that is split at all, and pieces of one head.
constexpr int kSplitMaxRows = kFwdPass128.max_items;
constexpr int kSplitMaxPieces = kSplitMaxRows + kFwdPass64.max_parts();
static_assert(kFwdPass64.max_items == kSplitMaxRows &&
                  kFwdPass64.max_parts() >= kFwdPass128.max_parts(),
              "bounds of both head dims");

// The runs of a tile within the limit fit kNoAllocScratchBytes; the order table
// and the split rows lie beside them.
constexpr size_t kNoAllocTableBytes =
    (kNoAllocMaxQBlocks > kSplitMaxPieces ? kNoAllocMaxQBlocks
                                          : kSplitMaxPieces) *
        sizeof(DevRow) +
    kFwdPass64.max_parts() * sizeof(DevSplit) + 4096;

struct PlanBuildParams {
  int32_t P, n, layout, causal;   // problem (partition length, partitions)
  int32_t nq, nkv, bm, bn;        // lists and the forward block shape
  int32_t nqb, nkbp;              // Q blocks of the tile, KV blocks per part
  split::Cut cut;
  int32_t m, mode;                // table entries, slot mapping
  DevRow* rows;                   // [m] in the scratch array
  DevRun* runs;                   // [<= 2 nqb nkv]
  DevSplit* splits;               // [split rows]
  int32_t* queue;                 // [8] lane counters, zeroed by the build
  int32_t q_idx[kNoAllocMaxList];
  int32_t kv_idx[kNoAllocMaxList];
};

// Device addresses of the scratch array and of the partial results' array
// (kNoAllocPartBytes) on the current device, looked up with
// hipGetSymbolAddress on the first call per device, then cached.
hipError_t noalloc_scratch(void** ptr, void** parts);

// Builds the forward work list and workgroup order of `p` (one workgroup).
hipError_t launch_fwd_plan_build(const PlanBuildParams& p, hipStream_t stream);

// Kernels with more than 64 KB of dynamic LDS need the limit raised once per
// kernel and device; this does it on the first launch on each device (ids
// below 64; higher ids set it on every launch).  Safe to call from several
// threads: the attribute set is idempotent and the flags are atomic.
template <auto Kern>
hipError_t ensure_dynamic_lds(size_t bytes) {
  static std::atomic<uint64_t> done{0};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const uint64_t bit = dev >= 0 && dev < 64 ? uint64_t{1} << dev : 0;
  if (bit != 0 && (done.load(std::memory_order_acquire) & bit) != 0)
    return hipSuccess;
  e = hipFuncSetAttribute(reinterpret_cast<const void*>(Kern),
                          hipFuncAttributeMaxDynamicSharedMemorySize,
                          static_cast<int>(bytes));
  if (e == hipSuccess && bit != 0)
    done.fetch_or(bit, std::memory_order_release);
  return e;
}

}  // namespace mesh_attn
