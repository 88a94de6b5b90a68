// Tile attention backward for gfx950 (MI355X): the per-pair gradient loop of
// Algorithm 3, summed over the tile.  Deterministic: every output element is
// owned by exactly one thread, no atomics.
//
// Two launches on the caller's stream, and a third where items were split, to
// sum their partial gradients:
//  1. prep:   D_i = <dO_i, O_i> and LSE_i * log2(e) for every (row, query
//     head), float32 (a row without a visible key gets +inf, so that its
//     probabilities exp2(s S - LSE) are 0); it also copies the work lists to
//     the workspace.
//  2. dK/dV:  one workgroup per (KV block of 128 keys, KV head), four waves of
//     32 keys.  It walks the KV block's runs of Q blocks (KV-major work list)
//     for every query head of the GQA group, in 64-row stages, and keeps dK,
//     dV in registers:
//     S = Q K^T,  P = exp(s S - LSE),  dP = dO V^T,  dS = P (dP - D),
//     dV += P^T dO,  dK += s dS^T Q.
//  3. dQ, in the same launch:  one workgroup per (Q block of 128 rows, query
//     head), four waves of 32 rows, walking the Q-major runs of KV blocks in
//     64-key stages:
//     S^T = K Q^T,  dP^T = V dO^T,  dS^T = P^T (dP^T - D),  dQ^T += s K^T dS^T.
//
// The stage tiles (Q and dO, or K and V: 64 rows x d) stream from HBM
// straight into LDS (buffer loads with the LDS-destination form), two stages
// deep with one barrier per stage.  Each tile is stored once, row-major, and
// read two ways: as rows (the A operand of the score MFMAs, 16-byte reads) and
// transposed (the B operand of dV / dK, the A operand of dQ) through the
// gfx950 LDS transpose read ds_read_b64_tr_b16.  One XOR swizzle of the
// 16-byte chunks serves both access patterns without bank conflicts.  As in
// the forward, the operand that feeds a score tile is read in the
// bit-2/3-swapped row order, so the probability and dS accumulators are
// already the k-contiguous operands of the next MFMA.

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "internal.h"
#include "tile_common.h"

namespace mesh_attn {
namespace {

using namespace dev;

constexpr int NT = kThreads;    // 256: four waves
constexpr int BQ = kBwdBM;      // 128
constexpr int BK = kBwdBN;      // 128
constexpr int SUB = kTileRows;  // 64 rows per LDS stage
constexpr float kLog2e = 1.4426950408889634f;

static_assert(BQ == 2 * SUB && BK == 2 * SUB, "two stages per block");

// ---------------------------------------------------------------------------
// 1. prep: delta and the log2-domain LSE
// ---------------------------------------------------------------------------
// The first plan_wgs workgroups copy the work lists of the two passes to the
// workspace, from pinned host memory or from the kernel's second argument.
constexpr size_t kBlobOffset =
    (sizeof(BwdParams) + alignof(PlanBlob) - 1) / alignof(PlanBlob) *
    alignof(PlanBlob);

template <int D>
__global__ __launch_bounds__(NT) void bwd_prep_kernel(BwdParams p, PlanBlob) {
  constexpr int LPI = D / 8;  // lanes per (row, head)
  const int plan_wgs = (p.plan_bytes / 16 + NT - 1) / NT;
  if (static_cast<int>(blockIdx.x) < plan_wgs) {
#if defined(__HIP_DEVICE_COMPILE__)
    const char* src =
        p.plan_src ? static_cast<const char*>(p.plan_src)
                   : (const char*)__builtin_amdgcn_kernarg_segment_ptr() +
                         kBlobOffset;
    const int i = blockIdx.x * NT + threadIdx.x;
    if (i < p.plan_bytes / 16)
      static_cast<f32x4*>(p.plan_dst)[i] =
          reinterpret_cast<const f32x4*>(src)[i];
#endif
    return;
  }
  const int64_t gid = int64_t{blockIdx.x - plan_wgs} * NT + threadIdx.x;
  const int64_t item = gid / LPI;  // row * hq + h
  const int sub = static_cast<int>(gid % LPI);
  const bool valid = item < p.rows_q * p.hq;
  float s = 0.f;
  if (valid) {
    const bf16x8 a = *reinterpret_cast<const bf16x8*>(p.o + item * D + sub * 8);
    const bf16x8 b =
        *reinterpret_cast<const bf16x8*>(p.d_o + item * D + sub * 8);
#pragma unroll
    for (int i = 0; i < 8; ++i)
      s = fmaf(static_cast<float>(a[i]), static_cast<float>(b[i]), s);
  }
#pragma unroll
  for (int off = LPI / 2; off > 0; off >>= 1) s += __shfl_xor(s, off);
  if (valid && sub == 0) {
    const int64_t row = item / p.hq;
    const int h = static_cast<int>(item - row * p.hq);
    const int64_t idx = int64_t{h} * p.rows_q + row;
    p.delta[idx] = s;
    const float lse = p.lse[idx];
    p.lse2[idx] = lse == -INFINITY ? INFINITY : lse * kLog2e;
  }
}

// ---------------------------------------------------------------------------
// Stage tiles: 64 rows x D bf16, row-major, 16-byte chunks XOR-swizzled.
// ---------------------------------------------------------------------------
template <int D>
struct StageTile {
  static constexpr int ROWB = 2 * D;        // bytes per row
  static constexpr int CPR = D / 8;         // 16-byte chunks per row
  static constexpr int RPI = 64 / CPR;      // rows per 1 KB wave load
  static constexpr int BYTES = SUB * ROWB;
  // Physical chunk of logical chunk c in row r is c ^ swz(r).  Row reads (16
  // lanes: 16 distinct rows, one chunk) need swz to be one-to-one on the 16
  // rows of a group; transpose reads (32 lanes: 4 rows x 4 chunks, or for
  // d = 64 two row pairs sharing the banks) need the rows of a quad to land
  // in different 4-chunk groups.  Both hold for these maps.
  __device__ static int swz(int r) {
    return D == 128 ? 4 * (r & 3) + ((r >> 2) & 3)
                    : 4 * ((r >> 1) & 1) + ((r >> 2) & 3);
  }
};

// Per-lane byte offsets into a stage tile.
template <int D>
struct TileAddr {
  using T = StageTile<D>;
  int row;         // row reads: row perm(li) (+32 t), chunk 2kk + lh
  int tr0, tr1;    // transpose reads, first and second half (+4 rows)

  __device__ void init(int lane) {
    const int li = lane & 31, lh = lane >> 5;
    {
      const int r = mfma_row_perm(li);
      row = r * T::ROWB + ((lh ^ T::swz(r)) * 16);
    }
    {
      // ds_read_b64_tr_b16: in 16-lane group g, lane s supplies row
      // 8*(g>>1) + s/4 (+4 for the second half, +16 per key step) at columns
      // 16*(g&1) + 4*(s%4) .. +3 of a 32-column chunk; lane l then holds
      // column l%32 of 8 consecutive rows (4 per half).
      const int g16 = lane >> 4, s16 = lane & 15;
      const int c16 = 2 * (g16 & 1) + ((s16 & 3) >> 1);
      const int r0 = 8 * (g16 >> 1) + (s16 >> 2);
      tr0 = r0 * T::ROWB + ((c16 ^ T::swz(r0)) * 16) + 8 * (s16 & 1);
      const int r1 = r0 + 4;
      tr1 = r1 * T::ROWB + ((c16 ^ T::swz(r1)) * 16) + 8 * (s16 & 1);
    }
  }
};

// Rows [row0, row0 + 64) of one head of a [rows][heads][D] bf16 tensor into a
// stage tile, shared by NW waves: wave wg loads rows wg*64/NW .. +64/NW with
// 1 KB loads.  Lane i of load j fills row wg*64/NW + j*RPI + i/CPR, physical
// chunk i%CPR, i.e. logical chunk (i%CPR) ^ swz(row).
template <int D, int NW = 4>
__device__ __forceinline__ void load_stage_tile(const uint16_t* base,
                                                int64_t row0, int heads,
                                                int head, char* tile, int wg,
                                                int lane) {
  using T = StageTile<D>;
  constexpr int RPW = SUB / NW;
  static_assert(RPW % T::RPI == 0, "whole loads per wave");
  const uint32_t row_bytes_g = static_cast<uint32_t>(heads) * D * 2;
  const rsrc_t r = make_rsrc(base + (row0 * heads + head) * D,
                             static_cast<uint32_t>(SUB) * row_bytes_g);
  const int lrow = lane / T::CPR, lchunk = lane % T::CPR;
  if constexpr (D == 128) {
    // swz(tr + lrow) = 4 (lrow & 3) + (tr / 4 & 3): one base, its chunk bits
    // XORed per load.
    const uint32_t base_off = lrow * row_bytes_g + (lchunk ^ (4 * lrow)) * 16;
#pragma unroll
    for (int j = 0; j < RPW / T::RPI; ++j) {
      const int tr = wg * RPW + j * T::RPI;  // first row of this load
      buffer_load16_lds(r, tile + tr * T::ROWB,
                        base_off ^ (16u * ((tr >> 2) & 3)), tr * row_bytes_g);
    }
  } else {
#pragma unroll
    for (int j = 0; j < RPW / T::RPI; ++j) {
      const int tr = wg * RPW + j * T::RPI;  // first row of this load
      const uint32_t voff =
          lrow * row_bytes_g + ((lchunk ^ T::swz(tr + lrow)) * 16);
      buffer_load16_lds(r, tile + tr * T::ROWB, voff, tr * row_bytes_g);
    }
  }
}

// 64 floats (one stage's rows of one head) into LDS, by one wave.
__device__ __forceinline__ void load_stage_floats(const float* src,
                                                  float* dst, int lane) {
  typedef __attribute__((address_space(3))) void lds_void;
  const rsrc_t r = make_rsrc(src, SUB * 4);
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void*)(dst), 4, lane * 4,
                                           0, 0, 0);
}

// A operand: rows perm(li) + 32*t of a tile, dims 16*kk + 8*lh .. +7.
template <int D>
__device__ __forceinline__ bf16x8 read_row_op(const char* tile, int addr,
                                              int t, int kk) {
  return *reinterpret_cast<const bf16x8*>(
      tile + (addr ^ (32 * kk)) + t * 32 * StageTile<D>::ROWB);
}

// Transposed operand: column 32*cc + l%32 of rows 16*ss + 8*lh .. +7.
template <int D>
__device__ __forceinline__ bf16x8 read_tr_op(const char* tile,
                                             const TileAddr<D>& a, int cc,
                                             int ss) {
  const char* b = tile + ss * 16 * StageTile<D>::ROWB;
  return join_bf16(lds_read_tr16(b + (a.tr0 ^ (64 * cc))),
                   lds_read_tr16(b + (a.tr1 ^ (64 * cc))));
}

// ---------------------------------------------------------------------------
// 2. dK / dV
// ---------------------------------------------------------------------------
// One gradient of a wave's 32 keys: dV (ROLE 0) or dK (ROLE 1, scaled).
// Accumulator register i of chunk c holds key row 8*(i/4) + 4*lh + i%4 of the
// wave's keys, dim 32*c + li.
// With accumulate, every old value is read before the first store, so the
// loads are issued back to back instead of one read-modify-write at a time.
template <int D, int ROLE>
__device__ __forceinline__ void write_keys(const BwdParams& p,
                                           const DevRow& pc, int hk, int kw,
                                           int li, int lh,
                                           const f32x16 (&acc)[D / 32]) {
  const int kvblk = pc.row;
  float* out = ROLE == 0 ? p.dv : p.dk;
  const float sc_out = ROLE == 0 ? 1.f : p.scale;
  if (pc.part >= 0) {
    const int64_t slot = int64_t{hk} * p.kvorder.parts + pc.part;
    float* po = p.kvparts + (slot * 2 + ROLE) * BK * D;
#pragma unroll
    for (int c = 0; c < D / 32; ++c)
#pragma unroll
      for (int i = 0; i < 16; ++i)
        po[(kw * 32 + 8 * (i >> 2) + 4 * lh + (i & 3)) * D + c * 32 + li] =
            acc[c][i] * sc_out;
    return;
  }
  auto index = [&](int c, int i) {
    const int64_t row =
        int64_t{kvblk} * BK + kw * 32 + 8 * (i >> 2) + 4 * lh + (i & 3);
    return (row * p.hkv + hk) * D + c * 32 + li;
  };
  f32x16 prev[D / 32];
#pragma unroll
  for (int c = 0; c < D / 32; ++c) zero(prev[c]);
  if (p.accumulate) {
#pragma unroll
    for (int c = 0; c < D / 32; ++c)
#pragma unroll
      for (int i = 0; i < 16; ++i) prev[c][i] = out[index(c, i)];
  }
#pragma unroll
  for (int c = 0; c < D / 32; ++c)
#pragma unroll
    for (int i = 0; i < 16; ++i)
      out[index(c, i)] = fmaf(acc[c][i], sc_out, prev[c][i]);
}

// Operand reads by LDS byte address: the stage's base is part of the address
// register, so that no XORed copies of it stay live over the loop.
typedef float f32x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ bf16x8 lds_frag(uint32_t a) {
  typedef __attribute__((address_space(3))) const bf16x8 T;
  return *(T*)a;
}
__device__ __forceinline__ f32x4 lds_f4(uint32_t a) {
  typedef __attribute__((address_space(3))) const f32x4 T;
  return *(T*)a;
}
__device__ __forceinline__ bf16x8 lds_tr(uint32_t a0, uint32_t a1, int imm) {
  typedef __attribute__((address_space(3))) s16x4 T;
  return join_bf16(__builtin_amdgcn_ds_read_tr16_b64_v4i16((T*)(a0 + imm)),
                   __builtin_amdgcn_ds_read_tr16_b64_v4i16((T*)(a1 + imm)));
}

// Order of a block of N MFMAs with R LDS operand reads each: the reads of
// AHEAD MFMAs in flight ahead of the MFMA that uses them.
template <int N, int R, int AHEAD>
__device__ __forceinline__ void pipeline_reads() {
  __builtin_amdgcn_sched_group_barrier(0x100, R * AHEAD, 0);
#pragma unroll
  for (int i = 0; i < N - AHEAD; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x100, R, 0);
  }
  __builtin_amdgcn_sched_group_barrier(0x008, AHEAD, 0);
}

// A wave holds everything of its 32 keys: K and V fragments and dK and dV
// accumulators, 192 registers at d = 128, 96 at d = 64, beside the scores.  At
// d = 128 that fits 256 registers (two workgroups per compute unit, 67 KB of
// LDS each) only because the addresses take five, S and dP use one tile of
// registers after the other and P is unpacked again for dS instead of kept in
// float32; d = 64 has room for both and fits 168 (three workgroups).  Before, eight waves in two roles
// passed P through LDS, one role a stage behind the other (two waves per SIMD).
// 8192 queries x 16384 keys x 32 heads, whole backward: d = 128 6730 us with
// the roles, 6533 without, 6450 with the operand reads two or three MFMAs ahead;
// d = 64 4073, 3574 and 3545.
template <int D>
struct DkdvLayout {
  static constexpr int TILE = StageTile<D>::BYTES;
  static constexpr int STAGE = 2 * TILE + 2 * SUB * 4;  // Q, dO, lse2, delta
  static constexpr int SMEM = 2 * STAGE;
};

template <int D>
__device__ __forceinline__ void dkdv_item(const BwdParams& p, char* smem,
                                           int block) {
  using L = DkdvLayout<D>;
  constexpr int ROWB = StageTile<D>::ROWB;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  const int li = lane & 31;
  const int lh = lane >> 5;
  const DevOrder& order = p.kvorder;
  const int slot = queued_slot(order.n_items, order.queue,
                               reinterpret_cast<int*>(smem + L::SMEM), block);
  if (slot < 0) return;
  // The whole item (its runs once per query head of the group), or a piece.
  int hk;
  const DevRow pc = load_slot(order, slot, p.hkv, 1, &hk);
  const int k_in_blk = wave * 32 + li;
  const int64_t kv_row = int64_t{pc.row} * BK + k_in_blk;

  bf16x8 kf[D / 16], vf[D / 16];
  load_frags<D>(kf, p.k, kv_row, p.hkv, hk, lh);
  load_frags<D>(vf, p.v, kv_row, p.hkv, hk, lh);
  f32x16 acc_v[D / 32], acc_k[D / 32];
#pragma unroll
  for (int c = 0; c < D / 32; ++c) {
    zero(acc_v[c]);
    zero(acc_k[c]);
  }

  if (pc.nblk > 0) {
    TileAddr<D> ta;
    ta.init(lane);
    // Stage cursor over (query head of the group, run, block in run, half).
    struct Cur {
      int g, r, off, s;
      DevRun run;
    };
    auto advance = [&](Cur c) {
      if (++c.s == 2) {
        c.s = 0;
        if (++c.off == c.run.nblk) {
          c.off = 0;
          if (++c.r == pc.run_e) {
            c.r = pc.run_b;
            ++c.g;
          }
          c.run = load_const(order.runs, c.r);
        }
      }
      return c;
    };
    auto issue = [&](const Cur& c, int buf) {
      char* base = smem + buf * L::STAGE;
      const int h = hk * p.group + c.g;
      const int64_t row0 = int64_t{c.run.blk0 + c.off} * BQ + c.s * SUB;
      load_stage_tile<D>(p.q, row0, p.hq, h, base, wave, lane);
      load_stage_tile<D>(p.d_o, row0, p.hq, h, base + L::TILE, wave, lane);
      float* f = reinterpret_cast<float*>(base + 2 * L::TILE);
      const int64_t at = int64_t{h} * p.rows_q + row0;
      if (wave == 0) load_stage_floats(p.lse2 + at, f, lane);
      if (wave == 1) load_stage_floats(p.delta + at, f + SUB, lane);
    };

    Cur cur{pc.walk, pc.run, pc.off, 0, load_const(order.runs, pc.run)};
    issue(cur, 0);
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk) {
      wait_for(kf[kk]);
      wait_for(vf[kk]);
    }
    wait_vmem();
    __syncthreads();
    int buf = 0;
    typedef __attribute__((address_space(3))) char lds_char;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_char*)smem;
    uint32_t ra = lds0 + ta.row, t0 = lds0 + ta.tr0, t1 = lds0 + ta.tr1;
    uint32_t fa = lds0 + 2 * L::TILE + lh * 32;
    for (int left = 2 * pc.nblk;;) {
      --left;
      const Cur nxt = advance(cur);
      if (left > 0) issue(nxt, buf ^ 1);
#pragma unroll
      for (int qt = 0; qt < 2; ++qt) {
        // S = Q K^T and dP = dO V^T: lane li owns key k_in_blk, register i
        // owns query 32*qt + acc_row(i, lh).  P = exp2(s S - LSE),
        // dS = P (dP - D).
        auto scores = [&](f32x16& x, const bf16x8 (&f)[D / 16], int tile) {
          zero(x);
#pragma unroll
          for (int kk = 0; kk < D / 16; ++kk)
            x = mfma32(lds_frag((ra ^ (32 * kk)) + tile + qt * 32 * ROWB),
                       f[kk], x);
        };
        auto mask = [&](f32x16& x) {
          if (cur.run.cls != 1) return;
          // key k of the block is hidden from query q of the run iff
          // k - q > delta + (offset of this stage in the run); the lane half's
          // share of the query index is on the limit's side.
          const int lim = k_in_blk - 8 * lh -
                          __builtin_amdgcn_readfirstlane(
                              cur.run.delta + cur.off * BQ + cur.s * SUB);
#pragma unroll
          for (int i = 0; i < 16; ++i)
            if (qt * 32 + acc_row(i, 0) < lim) x[i] = -INFINITY;
        };
        // LSE (j = 0) or D (j = 1) of queries 8*hh + 0..7 of the lane half.
        auto row_floats = [&](int j, int hh) {
          const uint32_t at = fa + 4 * (j * SUB + qt * 32 + hh * 16);
          const f32x4 lo = lds_f4(at), hi = lds_f4(at + 16);
          return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        };
        auto probs = [&](const f32x16& x, int hh) {
          const f32x8 lse = row_floats(0, hh);
          f32x8 e8;
#pragma unroll
          for (int e = 0; e < 8; ++e)
            e8[e] = exp2_fast(fmaf(x[hh * 8 + e], p.scale_log2, -lse[e]));
          return e8;
        };
        bf16x8 pf[2], ds[2];
        auto make_ds = [&](f32x8 e8, const f32x16& y, int hh) {
          const f32x8 dlt = row_floats(1, hh);
#pragma unroll
          for (int e = 0; e < 8; ++e) e8[e] *= y[hh * 8 + e] - dlt[e];
          ds[hh] = __builtin_convertvector(e8, bf16x8);
        };
        if constexpr (D == 64) {
          // Room for both score tiles: dS from P in float32.
          f32x16 x, y;
          scores(x, kf, 0);
          scores(y, vf, L::TILE);
          mask(x);
#pragma unroll
          for (int hh = 0; hh < 2; ++hh) {
            const f32x8 e8 = probs(x, hh);
            pf[hh] = __builtin_convertvector(e8, bf16x8);
            make_ds(e8, y, hh);
          }
        } else {
          f32x16 x;
          scores(x, kf, 0);
          pipeline_reads<D / 16, 1, 3>();
          mask(x);
#pragma unroll
          for (int hh = 0; hh < 2; ++hh) {
            pf[hh] = __builtin_convertvector(probs(x, hh), bf16x8);
            asm("" : "+v"(pf[hh]));  // unpack below instead of rounding again
          }
          __builtin_amdgcn_sched_barrier(0);
          scores(x, vf, L::TILE);
          pipeline_reads<D / 16, 1, 3>();
#pragma unroll
          for (int hh = 0; hh < 2; ++hh)
            make_ds(__builtin_convertvector(pf[hh], f32x8), x, hh);
          __builtin_amdgcn_sched_barrier(0);
        }
        // dV += P^T dO, dK += dS^T Q (scaled at the end).
#pragma unroll
        for (int c = 0; c < D / 32; ++c)
#pragma unroll
          for (int hh = 0; hh < 2; ++hh) {
            const uint32_t a0 = t0 ^ (64 * c), a1 = t1 ^ (64 * c);
            const int at = (2 * qt + hh) * 16 * ROWB;
            acc_v[c] = mfma32(pf[hh], lds_tr(a0, a1, L::TILE + at), acc_v[c]);
            acc_k[c] = mfma32(ds[hh], lds_tr(a0, a1, at), acc_k[c]);
          }
        if constexpr (D == 128) pipeline_reads<D / 8, 2, 2>();
      }
      if (left == 0) break;
      wait_vmem();
      lds_barrier();  // stage buf^1 landed; every wave is done with buf
      const int d = buf ? -L::STAGE : L::STAGE;
      ra += d;
      t0 += d;
      t1 += d;
      fa += d;
      buf ^= 1;
      cur = nxt;
    }
  }
  write_keys<D, 0>(p, pc, hk, wave, li, lh, acc_v);
  write_keys<D, 1>(p, pc, hk, wave, li, lh, acc_k);
}

// ---------------------------------------------------------------------------
// 3. dQ
// ---------------------------------------------------------------------------
template <int D>
struct DqLayout {
  static constexpr int TILE = StageTile<D>::BYTES;
  static constexpr int STAGE = 2 * TILE;  // K, V
  static constexpr int SMEM = 2 * STAGE;
};

template <int D>
__device__ __forceinline__ void dq_item(const BwdParams& p, char* smem,
                                        int block) {
  using L = DqLayout<D>;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  const int li = lane & 31;
  const int lh = lane >> 5;

  const DevOrder& order = p.qorder;
  const int slot = queued_slot(order.n_items, order.queue,
                               reinterpret_cast<int*>(smem + L::SMEM), block);
  if (slot < 0) return;
  // The whole item, or a piece of it.
  int h;
  const DevRow pc = load_slot(order, slot, p.hq, p.group, &h);
  const int qblk = pc.row;
  const int hk = h / p.group;
  const int q_in_blk = wave * 32 + li;
  const int64_t q_row = int64_t{qblk} * BQ + q_in_blk;

  bf16x8 qf[D / 16], dof[D / 16];
  load_frags<D>(qf, p.q, q_row, p.hq, h, lh);
  load_frags<D>(dof, p.d_o, q_row, p.hq, h, lh);
  const float lse2 = p.lse2[int64_t{h} * p.rows_q + q_row];
  const float dlt = p.delta[int64_t{h} * p.rows_q + q_row];

  f32x16 acc[D / 32];
#pragma unroll
  for (int cc = 0; cc < D / 32; ++cc) zero(acc[cc]);

  if (pc.nblk > 0) {
    TileAddr<D> ta;
    ta.init(lane);
    struct Cur {
      int r, off, s, left;  // left: stages from this one on
      DevRun run;
    };
    auto advance = [&](Cur c, bool* valid) {
      *valid = --c.left > 0;
      if (++c.s == 2) {
        c.s = 0;
        if (++c.off == c.run.nblk) {
          c.off = 0;
          ++c.r;
          if (*valid) c.run = load_const(order.runs, c.r);
        }
      }
      return c;
    };
    auto issue = [&](const Cur& c, int buf) {
      char* base = smem + buf * L::STAGE;
      const int64_t row0 = int64_t{c.run.blk0 + c.off} * BK + c.s * SUB;
      load_stage_tile<D>(p.k, row0, p.hkv, hk, base, wave, lane);
      load_stage_tile<D>(p.v, row0, p.hkv, hk, base + L::TILE, wave, lane);
    };

    Cur cur{pc.run, pc.off, 0, 2 * pc.nblk, load_const(order.runs, pc.run)};
    issue(cur, 0);
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk) {
      wait_for(qf[kk]);
      wait_for(dof[kk]);
    }
    wait_vmem();
    __syncthreads();
    int buf = 0;
    while (true) {
      bool has_next;
      const Cur nxt = advance(cur, &has_next);
      if (has_next) issue(nxt, buf ^ 1);

      const char* base = smem + buf * L::STAGE;
      const char* sk = base;
      const char* sv = base + L::TILE;

      // S^T = K Q^T, dP^T = V dO^T: lane li owns query q_in_blk, register i
      // owns key 32*kt + acc_row(i, lh) of the stage.
      f32x16 sc[2], dp[2];
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) {
        zero(sc[kt]);
        zero(dp[kt]);
#pragma unroll
        for (int kk = 0; kk < D / 16; ++kk) {
          sc[kt] = mfma32(read_row_op<D>(sk, ta.row, kt, kk), qf[kk], sc[kt]);
          dp[kt] = mfma32(read_row_op<D>(sv, ta.row, kt, kk), dof[kk], dp[kt]);
        }
      }
      {
        constexpr int NM = D / 4;  // one operand read per MFMA, 3 in flight
        __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);
#pragma unroll
        for (int i = 0; i < NM - 3; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, 3, 0);
      }
      if (cur.run.cls == 1) {
        const int lim = cur.run.delta - cur.off * BK - cur.s * SUB + q_in_blk;
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
          for (int i = 0; i < 16; ++i)
            if (kt * 32 + acc_row(i, lh) > lim) sc[kt][i] = -INFINITY;
      }
      bf16x8 dsb[4];
#pragma unroll
      for (int ss = 0; ss < 4; ++ss)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int kt = ss >> 1, i = (ss & 1) * 8 + e;
          const float pv = exp2_fast(fmaf(sc[kt][i], p.scale_log2, -lse2));
          dsb[ss][e] = static_cast<__bf16>(pv * (dp[kt][i] - dlt));
        }
      // dQ^T += K^T dS^T: the A operand K^T is read transposed from the K
      // row tile.
#pragma unroll
      for (int cc = 0; cc < D / 32; ++cc)
#pragma unroll
        for (int ss = 0; ss < 4; ++ss)
          acc[cc] = mfma32(read_tr_op<D>(sk, ta, cc, ss), dsb[ss], acc[cc]);
      {
        constexpr int NM = D / 8;  // two transpose reads per MFMA
        __builtin_amdgcn_sched_group_barrier(0x100, 6, 0);
#pragma unroll
        for (int i = 0; i < NM - 3; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, 3, 0);
      }

      if (!has_next) break;
      wait_vmem();
      lds_barrier();  // stage buf^1 landed; every wave is done with buf
      buf ^= 1;
      cur = nxt;
    }
  }

  // Register 4g+t of chunk cc holds dim 32cc + 8g + 4lh + t of query q_row.
  // With accumulate, all old values are read before the first store.
  if (pc.part >= 0) {
    const int64_t slot_p = int64_t{h} * order.parts + pc.part;
    float* po = p.qparts + (slot_p * BQ + q_in_blk) * D;
#pragma unroll
    for (int cc = 0; cc < D / 32; ++cc)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        f32x4 val;
#pragma unroll
        for (int t = 0; t < 4; ++t) val[t] = acc[cc][4 * g + t] * p.scale;
        *reinterpret_cast<f32x4*>(po + cc * 32 + g * 8 + lh * 4) = val;
      }
    return;
  }
  float* dst = p.dq + (q_row * p.hq + h) * D;
  f32x4 prev[D / 32][4];
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
            dst + cc * 32 + g * 8 + lh * 4);
  }
#pragma unroll
  for (int cc = 0; cc < D / 32; ++cc)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      f32x4 val;
#pragma unroll
      for (int t = 0; t < 4; ++t)
        val[t] = fmaf(acc[cc][4 * g + t], p.scale, prev[cc][g][t]);
      *reinterpret_cast<f32x4*>(dst + cc * 32 + g * 8 + lh * 4) = val;
    }
}

// Both passes in one launch, the dK/dV workgroups (the longer ones) first.
// They have the same shape (four waves; 256 registers and 67 and 64 KB of LDS at
// d = 128, 168 and 34 and 32 KB at d = 64), so dQ items fill the compute units
// that run out of dK/dV items and only one start and one end of a launch is
// paid: 72 -> 66 us for a 4K-token backward with d = 64, 930 -> 882 us for the
// four chunk tasks of a striped tile with d = 128.
template <int D>
__global__ __launch_bounds__(NT, D == 64 ? 3 : 2) void bwd_kernel(BwdParams p,
                                                                    int kv_wgs) {
  // Aligned so that XORs of an address's chunk bits do not reach its base.
  extern __shared__ __align__(256) char smem[];
  const int block = blockIdx.x;
  if (block < kv_wgs)
    dkdv_item<D>(p, smem, block);
  else
    dq_item<D>(p, smem, block - kv_wgs);
}

// ---------------------------------------------------------------------------
// Sum of the partial gradients of split items, in piece order (a fixed order,
// so the result stays deterministic).  A workgroup sums RPB rows of one
// tensor of one item, four dims a lane: 16-byte contiguous loads and stores.
// ---------------------------------------------------------------------------
template <int D>
struct SumLayout {
  static constexpr int LPR = D / 4;       // lanes per row
  static constexpr int RPB = NT / LPR;    // rows per workgroup
  static constexpr int GPT = 128 / RPB;   // workgroups per 128-row tensor
};

template <int D>
__global__ __launch_bounds__(NT) void bwd_sum_kernel(BwdParams p) {
  using L = SumLayout<D>;
  const int kv_wgs = p.kvorder.n_splits * p.hkv * 2 * L::GPT;
  const bool kv = static_cast<int>(blockIdx.x) < kv_wgs;
  const int wg = kv ? blockIdx.x : blockIdx.x - kv_wgs;
  const int si = wg / (kv ? 2 * L::GPT : L::GPT);
  const int role = kv ? wg / L::GPT % 2 : 0;  // 0: dV (or dQ), 1: dK
  const DevOrder& order = kv ? p.kvorder : p.qorder;
  const int head = si / order.n_splits;
  const DevSplit it = load_const(order.splits, si - head * order.n_splits);
  const int64_t part0 = int64_t{head} * order.parts + it.part;
  const int row = wg % L::GPT * L::RPB + threadIdx.x / L::LPR;
  const int col = threadIdx.x % L::LPR * 4;
  const int64_t stride = (kv ? 2 : 1) * 128 * D;  // floats per partial slot
  const float* src = (kv ? p.kvparts : p.qparts) + part0 * stride +
                     (role * 128 + row) * D + col;
  const int heads = kv ? p.hkv : p.hq;
  float* out = (kv ? (role ? p.dk : p.dv) : p.dq) +
               ((int64_t{it.row} * 128 + row) * heads + head) * D + col;
  // The stored value joins last, in one addition as with whole items: it may be
  // much larger than the partials, which must not be rounded to its last bit one
  // by one.
  f32x4 stored = {0.f, 0.f, 0.f, 0.f};
  if (p.accumulate) stored = *reinterpret_cast<const f32x4*>(out);
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  constexpr int B = 4;  // partials in flight
  for (int k0 = 0; k0 < it.nparts; k0 += B) {
    f32x4 x[B];
#pragma unroll
    for (int u = 0; u < B; ++u)
      x[u] = *reinterpret_cast<const f32x4*>(
          src + min(k0 + u, it.nparts - 1) * stride);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < B; ++u)
      if (k0 + u < it.nparts)
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[t] += x[u][t];
  }
#pragma unroll
  for (int t = 0; t < 4; ++t) acc[t] += stored[t];
  *reinterpret_cast<f32x4*>(out) = acc;
}

template <int D>
hipError_t launch(const BwdParams& p, const PlanBlob& blob,
                  hipStream_t stream) {
  const int64_t prep_threads = p.rows_q * p.hq * (D / 8);
  const int plan_wgs = (p.plan_bytes / 16 + NT - 1) / NT;
  const int prep_grid =
      plan_wgs + static_cast<int>((prep_threads + NT - 1) / NT);
  hipLaunchKernelGGL(bwd_prep_kernel<D>, dim3(prep_grid), dim3(NT), 0, stream,
                     p, blob);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int grid_kv = static_cast<int>(queued_launch_grid(p.kvorder.n_items));
  const int grid_q = static_cast<int>(queued_launch_grid(p.qorder.n_items));
  // LDS: + one int for the item slot of a queued workgroup.
  const size_t smem = std::max(DkdvLayout<D>::SMEM, DqLayout<D>::SMEM) + 16;
  e = ensure_dynamic_lds<bwd_kernel<D>>(smem);
  if (e != hipSuccess) return e;
  const int kv_wgs = (grid_kv + kNumXcd - 1) / kNumXcd * kNumXcd;
  hipLaunchKernelGGL(bwd_kernel<D>, dim3(kv_wgs + grid_q), dim3(NT), smem,
                     stream, p, kv_wgs);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int sums = (2 * p.kvorder.n_splits * p.hkv +
                    p.qorder.n_splits * p.hq) * SumLayout<D>::GPT;
  if (sums > 0) {
    hipLaunchKernelGGL(bwd_sum_kernel<D>, dim3(sums), dim3(NT), 0, stream, p);
    e = hipGetLastError();
  }
  return e;
}

}  // namespace

hipError_t launch_tile_bwd(const BwdParams& p, const PlanBlob& blob,
                           int head_dim, hipStream_t stream) {
  if (head_dim == 128) return launch<128>(p, blob, stream);
  if (head_dim == 64) return launch<64>(p, blob, stream);
  return hipErrorInvalidValue;
}

}  // namespace mesh_attn
