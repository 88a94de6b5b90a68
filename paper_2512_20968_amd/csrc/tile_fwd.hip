// Tile attention forward for gfx950 (MI355X).
//
// One workgroup computes one (Q block, query head) item: BM = 256 query rows,
// eight waves of 32 rows each.  It walks the Q block's runs of KV blocks
// (BN = 64 keys each) from the work list, so EMPTY blocks are never touched
// and only PARTIAL runs evaluate the causal mask (a wave-uniform branch).  For
// every KV block it forms scores, updates the online softmax of each row and
// accumulates P V -- the per-pair computation of Algorithm 2 with the
// online-softmax reducer applied inside the kernel (Section 2.2).
//
// Schedule: two-group ping-pong.  Waves 0-3 (group A) and 4-7 (group B)
// share the four SIMDs pairwise (wave w and w+4 on SIMD w % 4).  Per KV block
// each wave runs an MFMA phase X(n) -- the scores of block n+1 and
// O += V(n)^T P(n)^T -- and a VALU phase Y(n) -- mask, running max, rescale
// and the exponentials that make P(n+1).  Group B runs one phase behind
// group A and every phase ends at a workgroup barrier, so on each SIMD one
// wave's MFMAs always overlap the other wave's softmax.  Group B also issues
// the K/V loads, which makes both of its phases the longer ones of their
// slots, so its waves run at raised issue priority.  On launches with many
// items, the last items of each XCD's share are taken from per-XCD counters
// (queued_slot), so that faster XCDs take more of them.  On launches with few
// items (split.h) a workgroup computes one piece of an item's KV blocks and
// leaves a float32 partial result; fwd_combine_kernel folds them.  64 items of
// 1024 blocks (d = 128): 1350 us whole, 477 us in 256 pieces of 256 blocks;
// 64 causal items of 36 to 64 blocks: 107 us whole, 36 us split.
//
// Layout choices (64-wide wavefronts, v_mfma_f32_32x32x16_bf16):
//  * Scores are computed transposed, S^T = K Q^T (A = K rows from LDS,
//    B = Q columns held in registers for the whole item), so each lane owns
//    one query row and the row max / row sum are in-lane reductions plus one
//    exchange between the two half-waves.
//  * K rows are fed to the MFMA in an order that swaps bits 2 and 3 of the
//    row index, which leaves P^T in the accumulators already laid out as the
//    k-contiguous B operand of O^T += V^T P^T.
//  * K and V tiles stream from HBM straight into LDS (buffer loads with the
//    LDS-destination form, no staging registers), double buffered, rows
//    XOR-swizzled so every MFMA operand read is bank-conflict free.
//  * The V^T operand comes from the row-major V tile through the LDS
//    transpose read (ds_read_b64_tr_b16), two per MFMA.
//  * Softmax runs in the log2 domain with the scale folded into one FMA
//    before v_exp_f32.  The running max is exact, so a row's largest
//    probability is exactly 1 and its bf16 rounding is error-free.

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "internal.h"
#include "tile_common.h"

namespace mesh_attn {
namespace {

using namespace dev;

constexpr int BM = kFwdBM;  // 256
constexpr int BN = kFwdBN;  // 64
constexpr int NW = 8;       // waves per workgroup
constexpr int NT = NW * 64;
static_assert(BM == NW * 32, "one 32-row tile per wave");

template <int D>
struct FwdLayout {
  static constexpr int ROWB = 2 * D;         // bytes per K/V row
  static constexpr int CPR = D / 8;          // 16-byte chunks per row
  static constexpr int RPI = 64 / CPR;       // rows per 1 KB wave load
  static constexpr int RPW = BN / 4;         // rows each loading wave loads
  static constexpr int NLI = RPW / RPI;      // wave loads per tile
  static constexpr int TILE = BN * ROWB;     // bytes per K or V tile
  static constexpr int SMEM = 4 * TILE;      // K0, K1, V0, V1
  // XOR swizzles of the 16-byte chunk index, chosen so that the MFMA operand
  // reads below hit distinct LDS banks.
  __device__ static int kswz(int row) {
    return D == 128 ? (row & 15) : ((row >> 1) & 7);
  }
  __device__ static int vswz(int row) {
    return D == 128 ? 4 * (row & 3) : 4 * ((row >> 1) & 1);
  }
};

// Position in the flattened list of KV blocks of one Q block's runs, with the
// number of blocks left in this workgroup's piece of it.
struct Cursor {
  const DevRun* runs;
  DevRun run;
  int r, off, left;
};

// A KV block as the phases use it: its index in the tile's KV buffer (-1 past
// the end of the piece), the class of its run and the mask limit of the
// block's first query (key j is hidden from query i iff j - i > lim).
struct Blk {
  int idx, cls, lim;
  __device__ bool valid() const { return idx >= 0; }
};

__device__ __forceinline__ Blk block_at(const Cursor& c) {
  return Blk{c.left > 0 ? c.run.blk0 + c.off : -1, c.run.cls,
             c.run.delta - c.off * BN};
}

__device__ __forceinline__ Cursor next_block(Cursor c) {
  if (c.left <= 0) return c;
  --c.left;
  if (++c.off == c.run.nblk) {
    c.off = 0;
    ++c.r;
    if (c.left > 0) c.run = load_const(c.runs, c.r);
  }
  return c;
}

// Row order of a 32-key tile as fed to the MFMA: swap bits 2 and 3.
__device__ __forceinline__ int key_perm(int r) { return mfma_row_perm(r); }

// The order of the launch; a list that travels in the kernel's arguments is
// read there (the PlanBlob is the second argument).
constexpr size_t kBlobOffset =
    (sizeof(FwdParams) + alignof(PlanBlob) - 1) / alignof(PlanBlob) *
    alignof(PlanBlob);

__device__ __forceinline__ DevOrder order_of(const FwdParams& p) {
  DevOrder o = p.order;
#if defined(__HIP_DEVICE_COMPILE__)
  if (o.inline_list) {
    const char* blob =
        (const char*)__builtin_amdgcn_kernarg_segment_ptr() + kBlobOffset;
    o.rows = reinterpret_cast<const DevRow*>(blob);
    o.runs = reinterpret_cast<const DevRun*>(blob + o.off_runs);
    o.splits = reinterpret_cast<const DevSplit*>(blob + o.off_splits);
  }
#endif
  return o;
}

// Weights of the two-part online-softmax reducer (running accumulation: the
// stored pair and this call's): lse = M + log2(2^(old - M) + 2^(new - M)) with
// M the larger, O = w_old O_old + w_new O_new with w = 2^(lse_part - lse).
// Neither part sees a key: the stored O stays.  log2 units.
struct FoldWeights {
  float w_old, w_new, lse2;
};
__device__ __forceinline__ FoldWeights fold_weights(float old2, float new2) {
  const float mx = fmaxf(old2, new2);
  if (mx == -INFINITY) return {1.f, 0.f, new2};
  const float a = exp2_fast(old2 - mx), b = exp2_fast(new2 - mx);
  const float sum = a + b;
  return {a / sum, b / sum, mx + __builtin_amdgcn_logf(sum)};
}

// Four dims of a row of the result, the lanes of the row together: with
// `accumulate` (float32) folded into the stored pair.  All lanes of the row are
// in one wave and read the stored LSE before the first of them rewrites it
// (program order).
template <int D, bool OUT_F32>
__device__ __forceinline__ void store_folded(const FwdParams& p, int h,
                                             int64_t q_row, int col, f32x4 x,
                                             float lse2) {
  const int64_t lidx = int64_t{h} * p.rows_q + q_row;
  const int64_t oidx = (q_row * p.hq + h) * D + col;
  if constexpr (OUT_F32) {
    f32x4* dst = reinterpret_cast<f32x4*>(static_cast<float*>(p.o) + oidx);
    if (p.accumulate) {
      const FoldWeights w = fold_weights(p.lse[lidx] * 1.4426950408889634f,
                                         lse2);
      const f32x4 prev = *dst;
#pragma unroll
      for (int t = 0; t < 4; ++t) x[t] = fmaf(w.w_old, prev[t], w.w_new * x[t]);
      lse2 = w.lse2;
    }
    *dst = x;
  } else {
    bf16x4 val;
#pragma unroll
    for (int t = 0; t < 4; ++t) val[t] = static_cast<__bf16>(x[t]);
    *reinterpret_cast<bf16x4*>(static_cast<__bf16*>(p.o) + oidx) = val;
  }
  if (col == 0)
    p.lse[lidx] = lse2 == -INFINITY ? -INFINITY : lse2 * 0.69314718055994531f;
}

// Epilogue of one query row per lane pair (halves lh): O = acc / l, LSE =
// (m + log2 l) * ln 2, or a partial result.
template <int D, bool OUT_F32>
__device__ __forceinline__ void write_rows(const FwdParams& p,
                                           const DevOrder& order,
                                           const DevRow& item, int h,
                                           int64_t q_row, int q_in_blk, int lh,
                                           const f32x16 (&oacc)[D / 32],
                                           float m, float l) {
  const float lt = l + __shfl_xor(l, 32);
  const float inv = lt > 0.f ? 1.f / lt : 0.f;
  const float lse2 = lt > 0.f ? m + __builtin_amdgcn_logf(lt) : -INFINITY;
  if (item.part >= 0) {
    // A partial result: O normalised, float32, and the LSE in log2 units.  A
    // sum that is not a number stays so until the fold, whose result is then
    // the whole item's (O NaN, LSE -inf).
    const int64_t prow =
        int64_t{h * order.parts + item.part} * BM + q_in_blk;
    if (lh == 0) p.part_lse[prow] = lt == lt ? lse2 : lt;
#pragma unroll
    for (int cc = 0; cc < D / 32; ++cc)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        f32x4 x;
#pragma unroll
        for (int t = 0; t < 4; ++t) x[t] = oacc[cc][4 * g + t] * inv;
        *reinterpret_cast<f32x4*>(p.part_o + prow * D + cc * 32 + g * 8 +
                                  lh * 4) = x;
      }
    return;
  }
  const int64_t lidx = int64_t{h} * p.rows_q + q_row;
  // Running accumulation (float32 partials only): both lane halves of a row
  // read the stored LSE before the first half rewrites it (same wave, program
  // order).
  FoldWeights w{0.f, 1.f, lse2};
  if constexpr (OUT_F32) {
    if (p.accumulate)
      w = fold_weights(p.lse[lidx] * 1.4426950408889634f, lse2);
  }
  if (lh == 0)
    p.lse[lidx] =
        w.lse2 == -INFINITY ? -INFINITY : w.lse2 * 0.69314718055994531f;
  // O^T accumulator: register 4g+t of chunk cc holds dim 32cc + 8g + 4lh + t.
  const int64_t obase = (q_row * p.hq + h) * D;
  const float sc_new = inv * w.w_new;
  // Accumulating: every stored value is read before the first store, so the
  // loads are issued back to back.
  f32x4 prev[OUT_F32 ? D / 32 : 1][4];
  if constexpr (OUT_F32) {
#pragma unroll
    for (int cc = 0; cc < D / 32; ++cc)
#pragma unroll
      for (int g = 0; g < 4; ++g) prev[cc][g] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (p.accumulate) {
#pragma unroll
      for (int cc = 0; cc < D / 32; ++cc)
#pragma unroll
        for (int g = 0; g < 4; ++g)
          prev[cc][g] = *reinterpret_cast<const f32x4*>(
              static_cast<const float*>(p.o) + obase + cc * 32 + g * 8 +
              lh * 4);
    }
  }
#pragma unroll
  for (int cc = 0; cc < D / 32; ++cc)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int dim = cc * 32 + g * 8 + lh * 4;
      f32x4 x;
#pragma unroll
      for (int t = 0; t < 4; ++t) x[t] = oacc[cc][4 * g + t] * sc_new;
      if constexpr (OUT_F32) {
        f32x4* dst = reinterpret_cast<f32x4*>(static_cast<float*>(p.o) + obase +
                                              dim);
#pragma unroll
        for (int t = 0; t < 4; ++t) x[t] = fmaf(w.w_old, prev[cc][g][t], x[t]);
        *dst = x;
      } else {
        bf16x4 val;
#pragma unroll
        for (int t = 0; t < 4; ++t) val[t] = static_cast<__bf16>(x[t]);
        *reinterpret_cast<bf16x4*>(static_cast<__bf16*>(p.o) + obase + dim) =
            val;
      }
    }
}

// Head dim 128 (head dim 64 below).
template <int D, bool OUT_F32>
__global__ __launch_bounds__(NT, 1) void tile_fwd_kernel(FwdParams p,
                                                         PlanBlob) {
  static_assert(D == 128, "head dim 64 has a kernel of its own");
  using L = FwdLayout<D>;
  extern __shared__ __align__(16) char smem[];

  const int tid = threadIdx.x;
  // Wave index as a scalar (the compiler cannot infer that tid >> 6 is
  // uniform across the wave).
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = wave >> 2;   // 0: group A, 1: group B
  const int wg = wave & 3;     // wave within its group
  const int lane = tid & 63;
  const int li = lane & 31;
  const int lh = lane >> 5;

  // Item, or piece of one (order slot; see queued_static_slots).
  const DevOrder order = order_of(p);
  const int slot = queued_slot(order.n_items, order.queue,
                               reinterpret_cast<int*>(smem + L::SMEM), blockIdx.x);
  if (slot < 0) return;
  int h;
  const DevRow item = load_slot(order, slot, p.hq, p.group, &h);
  const int qblk = item.row;
  const int hk = h / p.group;
  Cursor c0;
  c0.runs = order.runs;
  c0.r = item.run;
  c0.off = item.off;
  c0.left = item.nblk;
  const int nblocks = c0.left;

  const int64_t q_row = int64_t{qblk} * BM + wave * 32 + li;
  const int q_in_blk = wave * 32 + li;

  // Q columns for the B operand: lane half lh holds dims 16kk + 8lh .. +7.
  bf16x8 qf[D / 16];
  load_frags<D>(qf, p.q, q_row, p.hq, h, lh);

  f32x16 oacc[D / 32];
#pragma unroll
  for (int cc = 0; cc < D / 32; ++cc) zero(oacc[cc]);
  float m = -INFINITY;  // reference max of scaled scores (log2 units)
  float l = 0.f;        // this lane's share of the row sum

  if (nblocks > 0) {
    c0.run = load_const(c0.runs, c0.r);
    // Direct global -> LDS staging, done by the four waves of group B.
    // Wave wg of the group fills rows wg*RPW .. +RPW of a tile with NLI
    // loads of 1 KB; lane i of load j takes row wg*RPW + j*RPI + i/CPR and
    // writes physical chunk i%CPR, i.e. the logical chunk
    // (i%CPR) ^ swizzle(row).
    const int64_t row_elems = int64_t{p.hkv} * D;  // elements per KV row
    const uint32_t row_bytes_g = static_cast<uint32_t>(row_elems * 2);
    const uint32_t blk_bytes = static_cast<uint32_t>(BN * row_elems * 2);
    // Every swizzled offset below has the form base ^ (stride * index): the
    // swizzle XORs a lane-dependent value into the chunk bits, and the loop
    // index only flips higher chunk bits that the row part leaves zero.  So
    // one base register per stream plus a v_xor per access replaces a
    // register per access.
    // Loads: lane i of load j reads logical chunk (i%CPR) ^ swizzle(row) of
    // row wg*RPW + j*RPI + i/CPR; for K that is kvo0 ^ (64 j), for V the
    // swizzle does not depend on j.
    const int lrow = lane / L::CPR;
    const uint32_t kvo0 =
        lrow * row_bytes_g + (((lane % L::CPR) ^ L::kswz(wg * L::RPW + lrow)) * 16);
    const uint32_t vvo0 =
        lrow * row_bytes_g + (((lane % L::CPR) ^ L::vswz(wg * L::RPW + lrow)) * 16);
    auto rsrc_of = [&](const uint16_t* base, int64_t blk) {
      return make_rsrc(base + (blk * BN * p.hkv + hk) * D, blk_bytes);
    };
    // LDS: K buffers 0, 1 then V buffers 0, 1; block j uses buffers j & 1.
    // One load round (the K tile of one block and the V tile of another) as
    // 2 NLI single loads, so that they can be spread over a phase.  A block
    // past the end gets an empty buffer range: its loads fetch nothing and
    // write zeros into a buffer that is free and never read.
    struct Round {
      rsrc_t rk, rv;
      char* kdst;
      char* vdst;
    };
    auto make_round = [&](const Blk& bk, const Blk& bv, int n) {
      Round rd;
      rd.rk = bk.valid() ? rsrc_of(p.k, bk.idx) : make_rsrc(p.k, 0);
      rd.rv = bv.valid() ? rsrc_of(p.v, bv.idx) : make_rsrc(p.v, 0);
      rd.kdst = smem + (n & 1) * L::TILE;
      rd.vdst = smem + (2 + ((n + 1) & 1)) * L::TILE;
      return rd;
    };
    auto load_part = [&](const Round& rd, int t) {  // t in [0, 2 NLI)
      const int j = t % L::NLI;
      const int row0 = wg * L::RPW + j * L::RPI;
      if (t < L::NLI)
        buffer_load16_lds(rd.rk, rd.kdst + row0 * L::ROWB, kvo0 ^ (64u * j),
                          row0 * row_bytes_g);
      else
        buffer_load16_lds(rd.rv, rd.vdst + row0 * L::ROWB, vvo0,
                          row0 * row_bytes_g);
    };
    auto load_k = [&](int64_t blk, int buf) {
      const rsrc_t rk = rsrc_of(p.k, blk);
#pragma unroll
      for (int j = 0; j < L::NLI; ++j) {
        const int row0 = wg * L::RPW + j * L::RPI;
        buffer_load16_lds(rk, smem + buf * L::TILE + row0 * L::ROWB,
                          kvo0 ^ (64u * j), row0 * row_bytes_g);
      }
    };
    auto load_v = [&](int64_t blk, int buf) {
      const rsrc_t rv = rsrc_of(p.v, blk);
#pragma unroll
      for (int j = 0; j < L::NLI; ++j) {
        const int row0 = wg * L::RPW + j * L::RPI;
        buffer_load16_lds(rv, smem + (2 + buf) * L::TILE + row0 * L::ROWB,
                          vvo0, row0 * row_bytes_g);
      }
    };
    // K operand read: row kt*32 + perm(li), dims 16kk + 8lh (logical chunk
    // 2kk + lh); the swizzle of such a row does not depend on kt, and the
    // byte offset is kra0 ^ (32 kk).
    int kra0;
    {
      const int prow = key_perm(li);
      kra0 = prow * L::ROWB + ((lh ^ L::kswz(prow)) * 16);
    }
    // V^T operand read (transpose): 16-lane group g, lane s reads row
    // 8*(g>>1) + s/4 (+16ss, +4 for the second half) at dims
    // 32cc + 16*(g&1) + 4*(s%4) .. +3; the swizzle of those rows depends on
    // s only, and the byte offset is vra0 ^ (64 cc).
    int vra0;
    {
      const int g16 = lane >> 4, s16 = lane & 15;
      const int vrow = 8 * (g16 >> 1) + (s16 >> 2);
      const int c16 = 2 * (g16 & 1) + ((s16 & 3) >> 1);
      vra0 = vrow * L::ROWB + ((c16 ^ L::vswz(vrow)) * 16) + 8 * (s16 & 1);
    }

    // S^T = K Q^T of one 64-key block from K buffer `buf`.
    auto scores = [&](f32x16 (&sc)[2], int buf) {
      const char* kb = smem + buf * L::TILE;
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) {
        zero(sc[kt]);
#pragma unroll
        for (int kk = 0; kk < D / 16; ++kk)
          sc[kt] = mfma32(*reinterpret_cast<const bf16x8*>(
                              kb + (kra0 ^ (32 * kk)) + kt * 32 * L::ROWB),
                          qf[kk], sc[kt]);
      }
      // Keep three operand reads in flight ahead of the MFMAs instead of
      // hoisting all of them (which would cost ~64 registers).
      constexpr int NM = D / 8;  // MFMAs in this block
      __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);
#pragma unroll
      for (int i = 0; i < NM - 3; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
      __builtin_amdgcn_sched_group_barrier(0x008, 3, 0);
    };
    // O^T += V^T P^T from V buffer `buf`; key step ss covers keys
    // 16ss + 8lh + 0..7.
    auto pv = [&](const bf16x8 (&pb)[4], int buf) {
      const char* vb = smem + (2 + buf) * L::TILE;
#pragma unroll
      for (int cc = 0; cc < D / 32; ++cc) {
#pragma unroll
        for (int ss = 0; ss < 4; ++ss) {
          const char* a0 = vb + (vra0 ^ (64 * cc)) + ss * 16 * L::ROWB;
          const bf16x8 a =
              join_bf16(lds_read_tr16(a0), lds_read_tr16(a0 + 4 * L::ROWB));
          oacc[cc] = mfma32(a, pb[ss], oacc[cc]);
        }
      }
      // Two transpose reads per MFMA, three MFMAs' worth in flight.
      constexpr int NM = D / 8;
      __builtin_amdgcn_sched_group_barrier(0x100, 6, 0);
#pragma unroll
      for (int i = 0; i < NM - 3; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
      }
      __builtin_amdgcn_sched_group_barrier(0x008, 3, 0);
    };
    // Softmax of one block's scores: causal mask (PARTIAL blocks: key j of
    // the run is hidden from query i of the Q block iff j - i > delta),
    // running max, rescale of O and l if some row of the wave has a new max,
    // then P = exp2(s S - m) into the bf16 B operand and the row sums.
    auto softmax = [&](f32x16 (&sc)[2], const Blk& bl, bf16x8 (&pb)[4],
                       auto&& hook) {
      if (bl.cls == 1) {
        const int lim = bl.lim + q_in_blk;
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
          for (int i = 0; i < 16; ++i)
            if (kt * 32 + acc_row(i, lh) > lim) sc[kt][i] = -INFINITY;
      }
      float mx = -INFINITY;
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int i = 0; i < 16; ++i) mx = fmaxf(mx, sc[kt][i]);
      mx = max_with_other_half(mx) * p.scale_log2;
      // Rescale O and l only when some row of the wave has a new maximum
      // (a wave-uniform branch).  Past the first few blocks of a row that is
      // rare, and the 4 * D / 2 multiplies would otherwise be the largest
      // VALU item of this phase after the exponentials.  A row whose maximum
      // is still -inf takes alpha = exp2(-inf) = 0 on 0-valued sums.
      const float m_new = fmaxf(m, mx);
      const float m_use = (m_new == -INFINITY) ? 0.f : m_new;
      if (__builtin_amdgcn_ballot_w64(m_new != m)) {
        const float alpha = exp2_fast(m - m_use);
        l *= alpha;
#pragma unroll
        for (int cc = 0; cc < D / 32; ++cc)
#pragma unroll
          for (int i = 0; i < 16; ++i) oacc[cc][i] *= alpha;
        m = m_new;
      }
      float rs[4];
#pragma unroll
      for (int ss = 0; ss < 4; ++ss) {
        hook(ss);
        float e8[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          e8[e] = exp2_fast(
              fmaf(sc[ss >> 1][(ss & 1) * 8 + e], p.scale_log2, -m_use));
          pb[ss][e] = static_cast<__bf16>(e8[e]);
        }
        rs[ss] = ((e8[0] + e8[1]) + (e8[2] + e8[3])) +
                 ((e8[4] + e8[5]) + (e8[6] + e8[7]));
      }
      l += (rs[0] + rs[1]) + (rs[2] + rs[3]);
    };

    // Prologue (all waves): K(0), V(0) and K(1) into LDS (group B loads),
    // then the scores and probabilities of block 0.
    const Blk b0 = block_at(c0);
    Cursor cu = next_block(c0);  // the block furthest ahead
    Blk bs = block_at(cu);          // block whose scores X(n) computes (n+1)
    if (grp == 1) {
      load_k(b0.idx, 0);
      load_v(b0.idx, 0);
      if (bs.valid()) load_k(bs.idx, 1);
    }
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk) wait_for(qf[kk]);
    wait_vmem();
    __syncthreads();
    bf16x8 pb[4];
    {
      f32x16 s0[2];
      scores(s0, 0);
      softmax(s0, b0, pb, [](int) {});
    }
    // Every wave has read K(0) before group B refills K buffer 0.
    __syncthreads();

    // Phase loops.  There are 2N slots (N = nblocks), each ending at a
    // workgroup barrier (an LDS-only barrier: group B's loads stay in flight
    // across the barrier of the slot that issues them).  Group A runs X(0) Y(0) X(1) ... X(N-1) and idles in
    // the last slot; group B idles in the first slot and then runs the same
    // sequence, one slot behind.  Group B issues the loads of K(n+2) and
    // V(n+1) in slot 2n and drains them at the end of slot 2n+1, so they are
    // in LDS by slot 2n+2, when A's X(n+1) first reads them; the buffers they
    // overwrite were last read in slots 2n-2 and 2n-1.
    f32x16 snx[2];
    if (grp == 0) {
      for (int n = 0; n < nblocks; ++n) {
        if (bs.valid()) scores(snx, (n + 1) & 1);
        pv(pb, n & 1);
        lds_barrier();
        if (bs.valid()) {
          softmax(snx, bs, pb, [](int) {});
          cu = next_block(cu);
          bs = block_at(cu);
        }
        lds_barrier();
      }
    } else {
      Blk bv = bs;  // V block to load next
      cu = next_block(cu);
      Blk bk = block_at(cu);  // K block to load next
      // Round n: K(n+2) and V(n+1), issued in slot 2n.  Issued as one burst
      // at the end of the softmax phase, the 2 NLI loads per wave held the
      // issuing waves up for several hundred cycles (measured: that phase
      // grew by about half); spread over the four exponential groups they
      // overlap the VALU work instead (about 5% faster overall).
      auto advance = [&]() {
        bv = bk;
        cu = next_block(cu);
        bk = block_at(cu);
      };
      {
        const Round rd = make_round(bk, bv, 0);
#pragma unroll
        for (int t = 0; t < 2 * L::NLI; ++t) load_part(rd, t);
        advance();
      }
      lds_barrier();
      // Group B's slots are the longer ones: its softmax phase also issues
      // the loads, and its MFMA phase runs beside group A's shorter softmax.
      // So its waves take issue priority over their group-A partners for the
      // whole loop (2-3 % faster than equal priority; raising it only for
      // the softmax phase gave half of that).
      __builtin_amdgcn_s_setprio(1);
      constexpr int PER = (2 * L::NLI) / 4;  // loads per exponential group
      static_assert(PER * 4 == 2 * L::NLI, "loads split evenly over 4 groups");
      for (int n = 0; n < nblocks; ++n) {
        if (bs.valid()) scores(snx, (n + 1) & 1);
        pv(pb, n & 1);
        wait_vmem();
        lds_barrier();
        // Block n+1 exists iff n + 1 < N; the last slot belongs to X(N-1)
        // and has no round after it.
        if (bs.valid()) {
          // Cursor updates (scalar code with branches) go first, so that the
          // compiler does not sink the exponentials below them, away from
          // the loads they are meant to hide.
          const Round rd = make_round(bk, bv, n + 1);
          const Blk cur = bs;
          bs = bv;
          advance();
          softmax(snx, cur, pb, [&](int ss) {
            // Keep the compiler from hoisting all loads to the phase start.
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < PER; ++t) load_part(rd, ss * PER + t);
          });
          lds_barrier();
        }
      }
      __builtin_amdgcn_s_setprio(0);
    }
  }

  write_rows<D, OUT_F32>(p, order, item, h, q_row, q_in_blk, lh, oacc, m, l);
}

// ---------------------------------------------------------------------------
// Head dim 64.  A 64-key block has half the MFMAs of d = 128 (16 per wave, 512
// cycles) and the same softmax (about 155 vector instructions per wave, 32 of
// them exponentials), so the vector unit bounds it.  The two ping-pong groups
// of d = 128 leave it idle whenever a wave waits on its own dependent
// instructions; four waves per SIMD do so less, and a wave of 32 rows fits 128
// registers at d = 64 (with 8 spilled, 36 bytes, all outside the key loop).  So
// two workgroups of eight waves share a compute unit,
// every wave loading its eighth of the K and V tiles of the next two blocks
// (64 KB per workgroup) before it computes two, one barrier per two blocks.
// 16384 rows x 32768 keys x 32 heads: 5141 us (856 TFLOP/s) with the ping-pong
// schedule, 4681 with one block per barrier here (vector unit busy in 75 % of
// the cycles, MFMA in 47 %, 1.91 GHz), 4508 (976 TFLOP/s) with two.
// ---------------------------------------------------------------------------
template <bool OUT_F32>
__global__ __launch_bounds__(NT, 4) void tile_fwd64_kernel(FwdParams p,
                                                           PlanBlob) {
  constexpr int D = 64;
  using L = FwdLayout<D>;
  extern __shared__ __align__(16) char smem[];
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  const int li = lane & 31;
  const int lh = lane >> 5;

  const DevOrder order = order_of(p);
  const int slot = queued_slot(order.n_items, order.queue,
                               reinterpret_cast<int*>(smem + 2 * L::SMEM), blockIdx.x);
  if (slot < 0) return;
  int h;
  const DevRow item = load_slot(order, slot, p.hq, p.group, &h);
  const int hk = h / p.group;
  Cursor cu;
  cu.runs = order.runs;
  cu.r = item.run;
  cu.off = item.off;
  cu.left = item.nblk;

  const int q_in_blk = wave * 32 + li;
  const int64_t q_row = int64_t{item.row} * BM + q_in_blk;
  bf16x8 qf[D / 16];
  load_frags<D>(qf, p.q, q_row, p.hq, h, lh);
  f32x16 oacc[D / 32];
#pragma unroll
  for (int cc = 0; cc < D / 32; ++cc) zero(oacc[cc]);
  float m = -INFINITY, l = 0.f;

  if (cu.left > 0) {
    cu.run = load_const(cu.runs, cu.r);
    const int64_t row_elems = int64_t{p.hkv} * D;
    const uint32_t row_bytes_g = static_cast<uint32_t>(row_elems * 2);
    const uint32_t blk_bytes = static_cast<uint32_t>(BN * row_elems * 2);
    // Loads: wave w fills rows 8w .. 8w + 7 of a tile, lane i row 8w + i/8,
    // physical chunk i%8.
    constexpr int RPW64 = BN / NW;  // 8 rows, one 1 KB load
    static_assert(RPW64 == L::RPI, "one load per wave and tile");
    const int lrow = wave * RPW64 + lane / L::CPR;
    const uint32_t kvo =
        lrow * row_bytes_g + (((lane % L::CPR) ^ L::kswz(lrow)) * 16);
    const uint32_t vvo =
        lrow * row_bytes_g + (((lane % L::CPR) ^ L::vswz(lrow)) * 16);
    auto load = [&](const Blk& b, int buf) {
      const int64_t at = (int64_t{b.idx} * BN * p.hkv + hk) * D;
      char* dst = smem + buf * 2 * L::TILE + wave * RPW64 * L::ROWB;
      buffer_load16_lds(make_rsrc(p.k + at, blk_bytes), dst, kvo, 0);
      buffer_load16_lds(make_rsrc(p.v + at, blk_bytes), dst + L::TILE, vvo, 0);
    };
    // Operand addresses as in the d = 128 kernel.
    int kra0, vra0;
    {
      const int prow = key_perm(li);
      kra0 = prow * L::ROWB + ((lh ^ L::kswz(prow)) * 16);
      const int g16 = lane >> 4, s16 = lane & 15;
      const int vrow = 8 * (g16 >> 1) + (s16 >> 2);
      const int c16 = 2 * (g16 & 1) + ((s16 & 3) >> 1);
      vra0 = vrow * L::ROWB + ((c16 ^ L::vswz(vrow)) * 16) + 8 * (s16 & 1);
    }

    // One block: scores, online softmax, O += P V (as the d = 128 phases).
    auto compute = [&](const Blk& cur, const char* kb) {
      const char* vb = kb + L::TILE;
      f32x16 sc[2];
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) {
        zero(sc[kt]);
#pragma unroll
        for (int kk = 0; kk < D / 16; ++kk)
          sc[kt] = mfma32(*reinterpret_cast<const bf16x8*>(
                              kb + (kra0 ^ (32 * kk)) + kt * 32 * L::ROWB),
                          qf[kk], sc[kt]);
      }
      if (cur.cls == 1) {
        const int lim = cur.lim + q_in_blk;
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
          for (int i = 0; i < 16; ++i)
            if (kt * 32 + acc_row(i, lh) > lim) sc[kt][i] = -INFINITY;
      }
      float mx = -INFINITY;
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int i = 0; i < 16; ++i) mx = fmaxf(mx, sc[kt][i]);
      mx = max_with_other_half(mx) * p.scale_log2;
      const float m_new = fmaxf(m, mx);
      const float m_use = (m_new == -INFINITY) ? 0.f : m_new;
      if (__builtin_amdgcn_ballot_w64(m_new != m)) {
        const float alpha = exp2_fast(m - m_use);
        l *= alpha;
#pragma unroll
        for (int cc = 0; cc < D / 32; ++cc)
#pragma unroll
          for (int i = 0; i < 16; ++i) oacc[cc][i] *= alpha;
        m = m_new;
      }
      float rs[4];
      bf16x8 pb[4];
#pragma unroll
      for (int ss = 0; ss < 4; ++ss) {
        float e8[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          e8[e] = exp2_fast(
              fmaf(sc[ss >> 1][(ss & 1) * 8 + e], p.scale_log2, -m_use));
          pb[ss][e] = static_cast<__bf16>(e8[e]);
        }
        rs[ss] = ((e8[0] + e8[1]) + (e8[2] + e8[3])) +
                 ((e8[4] + e8[5]) + (e8[6] + e8[7]));
      }
      l += (rs[0] + rs[1]) + (rs[2] + rs[3]);
#pragma unroll
      for (int cc = 0; cc < D / 32; ++cc) {
#pragma unroll
        for (int ss = 0; ss < 4; ++ss) {
          const char* a0 = vb + (vra0 ^ (64 * cc)) + ss * 16 * L::ROWB;
          const bf16x8 a =
              join_bf16(lds_read_tr16(a0), lds_read_tr16(a0 + 4 * L::ROWB));
          oacc[cc] = mfma32(a, pb[ss], oacc[cc]);
        }
      }
    };

    // Two blocks per barrier: the loads of the next two are in flight while
    // these two are computed.  Buffer pairs 0, 1 and 2, 3.
    Blk b0 = block_at(cu);
    cu = next_block(cu);
    Blk b1 = block_at(cu);
    load(b0, 0);
    if (b1.valid()) load(b1, 1);
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk) wait_for(qf[kk]);
    for (int pair = 0; b0.valid(); pair ^= 2) {
      // This wave's loads of the two blocks have landed; behind the barrier so
      // have all waves', and none still reads the other pair's buffers.
      wait_vmem();
      lds_barrier();
      cu = next_block(cu);
      const Blk n0 = block_at(cu);
      cu = next_block(cu);
      const Blk n1 = block_at(cu);
      if (n0.valid()) load(n0, pair ^ 2);
      if (n1.valid()) load(n1, (pair ^ 2) + 1);
      const char* kb = smem + pair * 2 * L::TILE;
      compute(b0, kb);
      if (b1.valid()) compute(b1, kb + 2 * L::TILE);
      b0 = n0;
      b1 = n1;
    }
  }
  write_rows<D, OUT_F32>(p, order, item, h, q_row, q_in_blk, lh, oacc, m, l);
}

// ---------------------------------------------------------------------------
// Tiles of a few short items (fwd_is_short): latency is all there is, and a
// workgroup of 256 rows walks its keys one block after the other on a few
// compute units.  Here a workgroup takes 32 rows and its waves take every
// S-th key block each (S = 8 waves at d = 64, 4 at d = 128), with K and V tiles
// of their own in LDS and no barrier; then they fold their results through
// LDS in wave order.  8 items of 8 blocks (d = 64, 64 workgroups): 15.3 us
// as 8 workgroups of 256 rows, 6.0 here.
// ---------------------------------------------------------------------------
template <int D>
struct ShortLayout {
  static constexpr int S = D == 64 ? 8 : 4;      // waves
  static constexpr int NT = S * 64;
  static constexpr int WAVE = 2 * FwdLayout<D>::TILE;  // K and V of one wave
  static constexpr int SMEM = S * WAVE;
  // A wave's result after the loop, in the same bytes: [32][D] floats with
  // rows padded against bank conflicts, then 32 maxima and 32 sums.
  static constexpr int ROWF = D + 4;
  static_assert((32 * ROWF + 64) * 4 <= WAVE, "result fits the wave's tiles");
};

template <int D, bool OUT_F32>
__global__ __launch_bounds__(ShortLayout<D>::NT) void tile_fwd_short_kernel(
    FwdParams p, PlanBlob) {
  using L = FwdLayout<D>;
  using SL = ShortLayout<D>;
  extern __shared__ __align__(16) char smem[];
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  const int li = lane & 31;
  const int lh = lane >> 5;
  const DevOrder order = order_of(p);
  int h;
  const DevRow item =
      load_slot(order, blockIdx.x / (BM / 32), p.hq, p.group, &h);
  const int hk = h / p.group;
  const int row0 = blockIdx.x % (BM / 32) * 32;  // within the Q block
  const int64_t q_row0 = int64_t{item.row} * BM + row0;

  bf16x8 qf[D / 16];
  load_frags<D>(qf, p.q, q_row0 + li, p.hq, h, lh);
  f32x16 oacc[D / 32];
#pragma unroll
  for (int cc = 0; cc < D / 32; ++cc) zero(oacc[cc]);
  float m = -INFINITY, l = 0.f;

  char* tile = smem + wave * SL::WAVE;
  Cursor cu;
  cu.runs = order.runs;
  cu.r = item.run;
  cu.off = item.off;
  cu.left = item.nblk;
  if (cu.left > 0) cu.run = load_const(cu.runs, cu.r);
  auto skip = [&](int n) {
    for (int i = 0; i < n; ++i) cu = next_block(cu);
  };
  skip(wave);
  const uint32_t row_bytes_g = static_cast<uint32_t>(p.hkv) * D * 2;
  int kra0, vra0;
  {
    const int prow = key_perm(li);
    kra0 = prow * L::ROWB + ((lh ^ L::kswz(prow)) * 16);
    const int g16 = lane >> 4, s16 = lane & 15;
    const int vrow = 8 * (g16 >> 1) + (s16 >> 2);
    const int c16 = 2 * (g16 & 1) + ((s16 & 3) >> 1);
    vra0 = vrow * L::ROWB + ((c16 ^ L::vswz(vrow)) * 16) + 8 * (s16 & 1);
  }
  for (Blk cur = block_at(cu); cur.valid();) {
    // The tiles' last readers are this wave's own MFMAs, whose operands have
    // arrived; then its own loads are all it waits for.
    const int64_t at = (int64_t{cur.idx} * BN * p.hkv + hk) * D;
    const rsrc_t rk = make_rsrc(p.k + at, BN * row_bytes_g);
    const rsrc_t rv = make_rsrc(p.v + at, BN * row_bytes_g);
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
    asm volatile("" ::: "memory");
#pragma unroll
    for (int j = 0; j < BN / L::RPI; ++j) {
      const int r = j * L::RPI + lane / L::CPR;
      buffer_load16_lds(rk, tile + j * L::RPI * L::ROWB,
                        r * row_bytes_g + ((lane % L::CPR) ^ L::kswz(r)) * 16,
                        0);
    }
#pragma unroll
    for (int j = 0; j < BN / L::RPI; ++j) {
      const int r = j * L::RPI + lane / L::CPR;
      buffer_load16_lds(rv, tile + L::TILE + j * L::RPI * L::ROWB,
                        r * row_bytes_g + ((lane % L::CPR) ^ L::vswz(r)) * 16,
                        0);
    }
    skip(SL::S);
    const Blk nxt = block_at(cu);
    wait_vmem();
    asm volatile("" ::: "memory");
    f32x16 sc[2];
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) {
      zero(sc[kt]);
#pragma unroll
      for (int kk = 0; kk < D / 16; ++kk)
        sc[kt] = mfma32(*reinterpret_cast<const bf16x8*>(
                            tile + (kra0 ^ (32 * kk)) + kt * 32 * L::ROWB),
                        qf[kk], sc[kt]);
    }
    if (cur.cls == 1) {
      const int lim = cur.lim + row0 + li;
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (kt * 32 + acc_row(i, lh) > lim) sc[kt][i] = -INFINITY;
    }
    float mx = -INFINITY;
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int i = 0; i < 16; ++i) mx = fmaxf(mx, sc[kt][i]);
    mx = max_with_other_half(mx) * p.scale_log2;
    const float m_new = fmaxf(m, mx);
    const float m_use = (m_new == -INFINITY) ? 0.f : m_new;
    const float alpha = exp2_fast(m - m_use);
    l *= alpha;
#pragma unroll
    for (int cc = 0; cc < D / 32; ++cc)
#pragma unroll
      for (int i = 0; i < 16; ++i) oacc[cc][i] *= alpha;
    m = m_new;
    bf16x8 pb[4];
#pragma unroll
    for (int ss = 0; ss < 4; ++ss) {
      float e8[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        e8[e] = exp2_fast(
            fmaf(sc[ss >> 1][(ss & 1) * 8 + e], p.scale_log2, -m_use));
        pb[ss][e] = static_cast<__bf16>(e8[e]);
      }
      l += ((e8[0] + e8[1]) + (e8[2] + e8[3])) +
           ((e8[4] + e8[5]) + (e8[6] + e8[7]));
    }
#pragma unroll
    for (int cc = 0; cc < D / 32; ++cc)
#pragma unroll
      for (int ss = 0; ss < 4; ++ss) {
        const char* a0 =
            tile + L::TILE + (vra0 ^ (64 * cc)) + ss * 16 * L::ROWB;
        const bf16x8 a =
            join_bf16(lds_read_tr16(a0), lds_read_tr16(a0 + 4 * L::ROWB));
        oacc[cc] = mfma32(a, pb[ss], oacc[cc]);
      }
    cur = nxt;
  }

  // Every wave's (O, m, l) of the 32 rows into its own LDS bytes, then the
  // fold: O = sum_w 2^(m_w - M) O_w / sum_w 2^(m_w - M) l_w.
  __builtin_amdgcn_s_waitcnt(0xC07F);  // its tile reads have arrived
  asm volatile("" ::: "memory");
  float* res = reinterpret_cast<float*>(tile);
#pragma unroll
  for (int cc = 0; cc < D / 32; ++cc)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      f32x4 x;
#pragma unroll
      for (int t = 0; t < 4; ++t) x[t] = oacc[cc][4 * g + t];
      *reinterpret_cast<f32x4*>(res + li * SL::ROWF + cc * 32 + g * 8 +
                                lh * 4) = x;
    }
  const float lt = l + __shfl_xor(l, 32);
  if (lh == 0) {
    res[32 * SL::ROWF + li] = m;
    res[32 * SL::ROWF + 32 + li] = lt;
  }
  __syncthreads();
  constexpr int LPR = D / 4;                 // lanes per row, four dims each
  constexpr int RPP = SL::NT / LPR;          // rows per pass
  const int col = tid % LPR * 4;
#pragma unroll
  for (int pass = 0; pass < 32 / RPP; ++pass) {
    const int r = pass * RPP + tid / LPR;
    auto part = [&](int w) {
      return reinterpret_cast<const float*>(smem + w * SL::WAVE);
    };
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < SL::S; ++w)
      M = fmaxf(M, part(w)[32 * SL::ROWF + r]);
    const float mu = M == -INFINITY ? 0.f : M;
    float sum = 0.f;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < SL::S; ++w) {
      const float a = exp2_fast(part(w)[32 * SL::ROWF + r] - mu);
      sum = fmaf(a, part(w)[32 * SL::ROWF + 32 + r], sum);
      const f32x4 x =
          *reinterpret_cast<const f32x4*>(part(w) + r * SL::ROWF + col);
#pragma unroll
      for (int t = 0; t < 4; ++t) acc[t] = fmaf(a, x[t], acc[t]);
    }
    const float inv = sum > 0.f ? 1.f / sum : 0.f;
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[t] *= inv;
    const float lse2 =
        sum > 0.f ? M + __builtin_amdgcn_logf(sum) : -INFINITY;
    store_folded<D, OUT_F32>(p, h, q_row0 + r, col, acc, lse2);
  }
}

// ---------------------------------------------------------------------------
// Fold of the partial results of split items (the online-softmax reducer, in
// piece order): one workgroup per 256 / (D / 4) rows of an item, a lane per
// four dims of a row, so that loads and stores are 16 bytes and contiguous.
// Bound by memory: 256 partials of 256 x 128 (34 MB) in 7-9 us.
// ---------------------------------------------------------------------------
constexpr int NTC = 256;

template <int D, bool OUT_F32>
__global__ __launch_bounds__(NTC) void fwd_combine_kernel(FwdParams p,
                                                          PlanBlob) {
  constexpr int LPR = D / 4;             // lanes per row
  constexpr int RPB = NTC / LPR;         // rows per workgroup
  constexpr int GPI = BM / RPB;          // workgroups per item
  const DevOrder order = order_of(p);
  const int si = blockIdx.x / GPI, h = si / order.n_splits;
  const DevSplit it = load_const(order.splits, si - h * order.n_splits);
  const int64_t part0 = int64_t{h} * order.parts + it.part;
  const int row = (blockIdx.x % GPI) * RPB + threadIdx.x / LPR;
  const int sub = threadIdx.x % LPR;
  const int64_t q_row = int64_t{it.row} * BM + row;
  float M = -INFINITY, S = 0.f;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  auto fold = [&](const f32x4& x, float lse) {
    const float mn = fmaxf(M, lse);
    const float mu = mn == -INFINITY ? 0.f : mn;
    const float r = exp2_fast(M - mu), w = exp2_fast(lse - mu);
    S = fmaf(S, r, w);
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[t] = fmaf(w, x[t], acc[t] * r);
    M = mn;
  };
  constexpr int B = 4;  // partials in flight
  for (int k0 = 0; k0 < it.nparts; k0 += B) {
    f32x4 x[B];
    float lv[B];
#pragma unroll
    for (int u = 0; u < B; ++u) {
      const int k = min(k0 + u, it.nparts - 1);
      const int64_t prow = (part0 + k) * BM + row;
      x[u] = *reinterpret_cast<const f32x4*>(p.part_o + prow * D + sub * 4);
      lv[u] = p.part_lse[prow];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < B; ++u)
      if (k0 + u < it.nparts) fold(x[u], lv[u]);
  }
  const float inv = S > 0.f ? 1.f / S : 0.f;
#pragma unroll
  for (int t = 0; t < 4; ++t) acc[t] *= inv;
  store_folded<D, OUT_F32>(
      p, h, q_row, sub * 4, acc,
      S > 0.f ? M + __builtin_amdgcn_logf(S) : -INFINITY);
}

template <int D, bool F32>
hipError_t launch(const FwdParams& p, const PlanBlob& blob,
                  hipStream_t stream) {
  const int grid = static_cast<int>(queued_launch_grid(p.order.n_items));
  hipError_t e = hipSuccess;
  if (p.order.is_short) {
    using SL = ShortLayout<D>;
    e = ensure_dynamic_lds<tile_fwd_short_kernel<D, F32>>(SL::SMEM);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((tile_fwd_short_kernel<D, F32>),
                       dim3(p.order.n_items * (BM / 32)), dim3(SL::NT),
                       SL::SMEM, stream, p, blob);
    return hipGetLastError();
  }
  // + the item slot; head dim 64 keeps four blocks in LDS, 128 two.
  const size_t smem = (D == 64 ? 2 : 1) * FwdLayout<D>::SMEM + 16;
  constexpr auto kernel = [] {
    if constexpr (D == 64)
      return tile_fwd64_kernel<F32>;
    else
      return tile_fwd_kernel<D, F32>;
  }();
  e = ensure_dynamic_lds<kernel>(smem);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kernel, dim3(grid), dim3(NT), smem, stream, p, blob);
  e = hipGetLastError();
  if (e != hipSuccess || p.order.n_splits == 0) return e;
  constexpr int GPI = BM / (NTC / (D / 4));
  hipLaunchKernelGGL((fwd_combine_kernel<D, F32>),
                     dim3(p.order.n_splits * p.hq * GPI), dim3(NTC), 0, stream,
                     p, blob);
  return hipGetLastError();
}

// 16 bytes a lane.
__global__ __launch_bounds__(NTC) void plan_copy_kernel(f32x4* dst,
                                                        const f32x4* src,
                                                        int n) {
  const int i = blockIdx.x * NTC + threadIdx.x;
  if (i < n) dst[i] = src[i];
}

}  // namespace

hipError_t launch_plan_copy(void* dst, const void* src, size_t bytes,
                            hipStream_t stream) {
  const int n = static_cast<int>(bytes / 16);
  hipLaunchKernelGGL(plan_copy_kernel, dim3((n + NTC - 1) / NTC), dim3(NTC), 0,
                     stream, static_cast<f32x4*>(dst),
                     static_cast<const f32x4*>(src), n);
  return hipGetLastError();
}

hipError_t launch_tile_fwd(const FwdParams& p, const PlanBlob& blob,
                           int head_dim, bool out_f32, hipStream_t stream) {
  if (head_dim == 128)
    return out_f32 ? launch<128, true>(p, blob, stream)
                   : launch<128, false>(p, blob, stream);
  if (head_dim == 64)
    return out_f32 ? launch<64, true>(p, blob, stream)
                   : launch<64, false>(p, blob, stream);
  return hipErrorInvalidValue;
}

}  // namespace mesh_attn
