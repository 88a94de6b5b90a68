// Host-side builder of a pass's work list in the kernels' form: the order
// table, the runs and the split rows of one orientation of a tile.
//
// All heads of a tile have the same work, so the table lists the pieces of one
// head in rank order and a workgroup finds its piece and head from its slot
// (plan_slot in split.h).  Runs follow the canonical work list (the causal
// rule of Section 3.7 per block pair, KV or Q partitions in list order, EMPTY
// dropped), except that FULL runs that continue each other in the tile's
// buffer are one run.  Positions grow linearly with the row inside a
// partition, so the run boundaries have closed forms.
//
// The builder allocates nothing: it fills arrays of the caller and says so if
// they are too small.
#pragma once

#include <algorithm>

#include "internal.h"
#include "mesh_attn.h"

namespace mesh_attn {
namespace plan {

// The rows of each partition a buffer holds: `len` consecutive local rows
// starting at local row `off` (the whole partition, or one GOO chunk of it).
struct Slice {
  int64_t len, off;
};

// Global position of token `row` of partition `part` (Section 3.7 layouts).
// Within a partition positions grow with the row under both layouts, so a
// block's first and last rows hold its extreme positions.
inline int64_t token_pos(const ma_problem_t* p, int32_t part, int64_t row) {
  return p->layout == MA_LAYOUT_STRIPED
             ? row * p->num_partitions + part
             : int64_t{part} * p->partition_len + row;
}

// Mask offset of a (query block, key run) pair in rows: key row k0 + j is
// hidden from query row q0 + i iff j - i > offset.  Contiguous: the position
// difference q0 - k0 across partitions.  Striped: position (row * n + part),
// so key after query iff (j - i) * n > (q0 - k0) * n + (qp - kp), i.e. iff
// j - i > (q0 - k0) + floor((qp - kp) / n), and |qp - kp| < n.
inline int64_t mask_offset(const ma_problem_t* p, int32_t qp, int64_t q0,
                           int32_t kp, int64_t k0) {
  if (p->layout == MA_LAYOUT_STRIPED) return (q0 - k0) + (qp >= kp ? 0 : -1);
  return token_pos(p, qp, q0) - token_pos(p, kp, k0);
}

// One orientation of a tile.  Side A blocks (bm_a rows) own the workgroups,
// side B blocks (bm_b rows) are walked, `walks` times.  a_is_q: side A is the
// query side.  `heads` heads own workgroups, `group` of them per KV head.
// pass: how long items may be split, null to leave them whole; forward: its
// items may be short ones (fwd_is_short).
struct Side {
  const ma_problem_t* p;
  const int32_t* a_idx;
  int32_t na, bm_a;
  Slice sa;
  const int32_t* b_idx;
  int32_t nb, bm_b;
  Slice sb;
  bool a_is_q;
  int32_t heads, group, walks;
  const split::Pass* pass;
  bool forward;

  int32_t rows() const { return na * static_cast<int32_t>(sa.len / bm_a); }
};

// What the builder fills: caller's arrays and their capacities, `work` one
// entry per row of side A.
struct Arrays {
  DevRow* rows;
  int64_t cap_rows;
  DevRun* runs;
  int64_t cap_runs;
  DevSplit* splits;
  int64_t cap_splits;
  int32_t* work;
};

struct Built {
  int32_t m = 0, n_runs = 0, n_splits = 0;  // table entries, runs, split rows
  int32_t parts = 0;                        // partials per head
  int32_t mode = 0;
  bool is_short = false;
};

// Blocks kb of [0, n) with base + kb * step <= x.
inline int64_t count_le(int64_t base, int64_t step, int64_t x, int64_t n) {
  return x < base ? 0 : std::min(n, (x - base) / step + 1);
}

// FULL and PARTIAL blocks of side B's list entry b against row block (part,
// row0) of side A: an ascending pair of ranges [begin, end) with classes.
struct PairRuns {
  int64_t begin[2], end[2];
  int cls[2];
};
inline PairRuns pair_runs(const Side& s, int32_t a_part, int64_t a_row0,
                          int32_t b_part) {
  const int64_t n = s.sb.len / s.bm_b;
  if (!s.p->causal) return {{0, n}, {n, n}, {MA_CLS_FULL, MA_CLS_PARTIAL}};
  const int64_t a0 = token_pos(s.p, a_part, a_row0);
  const int64_t a1 = token_pos(s.p, a_part, a_row0 + s.bm_a - 1);
  const int64_t b0 = token_pos(s.p, b_part, s.sb.off);
  const int64_t b1 = token_pos(s.p, b_part, s.sb.off + s.bm_b - 1);
  const int64_t step = token_pos(s.p, 0, s.bm_b);
  if (s.a_is_q) {
    // FULL: the block's last key is at or before the first query; not EMPTY:
    // its first key is at or before the last query.
    const int64_t full = count_le(b1, step, a0, n);
    const int64_t vis = count_le(b0, step, a1, n);
    return {{0, full}, {full, vis}, {MA_CLS_FULL, MA_CLS_PARTIAL}};
  }
  // EMPTY: the block's last query is before the first key; not yet FULL: its
  // first query is before the last key.
  const int64_t empty = count_le(b1, step, a0 - 1, n);
  const int64_t below = count_le(b0, step, a1 - 1, n);
  return {{empty, below}, {below, n}, {MA_CLS_PARTIAL, MA_CLS_FULL}};
}

// Builds the plan of one side; false if an array is too small.
inline bool build(const Side& s, const Arrays& out, Built* built) {
  Built b;
  const int32_t rows = s.rows();
  const int32_t nab = static_cast<int32_t>(s.sa.len / s.bm_a);
  const int32_t nbb = static_cast<int32_t>(s.sb.len / s.bm_b);
  if (rows > out.cap_rows) return false;
  // Runs of every row; the table's first `rows` entries hold their ranges
  // until the pieces are known.
  for (int32_t r = 0; r < rows; ++r) {
    const int32_t part = s.a_idx[r / nab];
    const int64_t row0 = s.sa.off + int64_t{r % nab} * s.bm_a;
    const int32_t first = b.n_runs;
    int64_t work = 0;
    for (int32_t e = 0; e < s.nb; ++e) {
      const PairRuns pr = pair_runs(s, part, row0, s.b_idx[e]);
      for (int i = 0; i < 2; ++i) {
        const int64_t n = pr.end[i] - pr.begin[i];
        if (n <= 0) continue;
        work += n;
        const int32_t blk0 = static_cast<int32_t>(e * nbb + pr.begin[i]);
        DevRun* last = b.n_runs > first ? &out.runs[b.n_runs - 1] : nullptr;
        if (last && last->cls == MA_CLS_FULL && pr.cls[i] == MA_CLS_FULL &&
            last->blk0 + last->nblk == blk0) {
          last->nblk += static_cast<int32_t>(n);
          continue;
        }
        if (b.n_runs == out.cap_runs) return false;
        const int64_t b_row0 = s.sb.off + pr.begin[i] * s.bm_b;
        const int64_t delta =
            s.a_is_q ? mask_offset(s.p, part, row0, s.b_idx[e], b_row0)
                     : mask_offset(s.p, s.b_idx[e], b_row0, part, row0);
        out.runs[b.n_runs++] =
            DevRun{blk0, static_cast<int32_t>(n), pr.cls[i],
                   static_cast<int32_t>(delta)};
      }
    }
    out.work[r] = static_cast<int32_t>(work * s.walks);
    out.rows[r].run_b = first;
    out.rows[r].run_e = b.n_runs;
  }
  b.is_short = s.forward &&
               fwd_is_short(int64_t{rows} * s.heads,
                            *std::max_element(out.work, out.work + rows),
                            s.p->head_dim);
  const split::Cut cut =
      s.pass && !b.is_short
          ? split::choose(out.work, rows, s.heads, *s.pass)
          : split::Cut{};
  for (int32_t r = 0; r < rows; ++r) {
    const int32_t n = split::num_pieces(cut, r, out.work[r]);
    b.m += n;
    if (n == 1) continue;
    if (b.n_splits == out.cap_splits) return false;
    out.splits[b.n_splits++] = DevSplit{r, b.parts, n};
    b.parts += n;
  }
  if (b.m > out.cap_rows) return false;
  // Pieces, last row first so that a row's range is read before its place in
  // the table is overwritten.
  int32_t at = b.m, part = b.parts;
  for (int32_t r = rows - 1; r >= 0; --r) {
    const int32_t run_b = out.rows[r].run_b, run_e = out.rows[r].run_e;
    const int32_t w = out.work[r], n = split::num_pieces(cut, r, w);
    at -= n;
    if (n > 1) part -= n;
    int32_t run = run_b, off = 0, walk = 0;
    for (int32_t j = 0; j < n; ++j) {
      const int32_t len =
          split::piece_begin(w, n, j + 1) - split::piece_begin(w, n, j);
      while (len > 0 && off >= out.runs[run].nblk) {
        off -= out.runs[run++].nblk;
        if (run == run_e) {
          run = run_b;
          ++walk;
        }
      }
      out.rows[at + j] = DevRow{r,    run,   off,   len, n > 1 ? part + j : -1,
                                walk, run_b, run_e, j,   0};
      off += len;
    }
  }
  // Rank order: longest first, or in one round of a split tile by piece index
  // (`before` holds it until the ranks are known).
  b.mode = split_mode(int64_t{b.m} * s.heads, cut.c > 0,
                      s.heads / s.group % kNumXcd == 0, cut.slots);
  const bool by_len = b.mode != kModeOneRound;
  auto key = [&](const DevRow& x) { return by_len ? -x.nblk : x.before; };
  std::sort(out.rows, out.rows + b.m, [&](const DevRow& x, const DevRow& y) {
    if (key(x) != key(y)) return key(x) < key(y);
    if (x.row != y.row) return x.row < y.row;
    return x.before < y.before;
  });
  for (int32_t i = 0, j; i < b.m; i = j) {
    for (j = i + 1; j < b.m && key(out.rows[j]) == key(out.rows[i]);) ++j;
    // `before` of the entries behind i is still their piece index.
    for (int32_t k = i; k < j; ++k) out.rows[k].same = j - i;
    for (int32_t k = i; k < j; ++k) out.rows[k].before = i;
  }
  *built = b;
  return true;
}

}  // namespace plan
}  // namespace mesh_attn
