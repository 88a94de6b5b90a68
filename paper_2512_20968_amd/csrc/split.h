// Splitting of long work items over the blocks they walk, for launches with
// too few items to fill the chip evenly.
//
// An item is one (block row, head) pair of a pass; every head has the same
// work w[0..n) (blocks per row).  An item may be cut into equal pieces that
// different workgroups compute as partial results and a second kernel folds.
// The number of pieces of a row depends on its work alone, so all heads are
// cut alike, the pieces of the rows of one KV head cover the same key ranges
// (their workgroups share them in L2) and the XCD lanes stay even.  Integer
// arithmetic on the work list only: the host and the device-side list builder
// cut alike, and a tile gives the same bits from both.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mesh_attn {
namespace split {

// A pass as the cut sees it; times in blocks of one of its workgroups.
struct Pass {
  int32_t slots;      // workgroups that run at once
  int32_t max_items;  // tiles of more items than this are never split: the
                      // longest first order leaves at most a fraction of a
                      // round of many idle
  int32_t overhead;   // a workgroup's start and end (work list, first tiles,
                      // fragments, epilogue)
  int32_t min_piece;  // shortest piece worth a workgroup and a partial result;
                      // items of at most two such pieces stay whole
  int32_t fold;       // launch of the kernel that folds the partials
  int32_t fold_rate;  // partials written and read back per block
  // Where two workgroups share a compute unit, whole items that have one each
  // run faster than their slots say: alone blocks per 100 and alone_overhead.
  int32_t alone = 0, alone_overhead = 0;
  // The pass with fewer slots, where it shares its launch with another one: a
  // tile that is left whole for all of its slots is looked at again for these.
  const Pass* beside = nullptr;
  // Most partial results a pass holds.
  __host__ __device__ constexpr int32_t max_parts() const { return 2 * slots; }
};

// Rows [0, whole) of every head stay whole, the others are cut into pieces of
// at most c blocks, for a round of `slots` workgroups; c = 0: nothing is cut.
struct Cut {
  int32_t c = 0, whole = 0, slots = 0;
};

__host__ __device__ inline int32_t num_pieces(const Cut& s, int32_t row,
                                              int32_t w) {
  return s.c > 0 && row >= s.whole && w > s.c ? (w + s.c - 1) / s.c : 1;
}

// First block of piece j of n: w * j / n, without 64-bit division (j and n are at
// most a few thousand).
__host__ __device__ inline int32_t piece_begin(int32_t w, int32_t n,
                                               int32_t j) {
  return w / n * j + w % n * j / n;
}

// Partial results a tile may need, from its sizes alone: `items` items of at
// most `max_work` blocks.  Never less than what choose() gives.
inline int64_t parts_bound(int64_t items, int64_t max_work,
                           const Pass& ps) {
  if (items > ps.max_items || max_work <= 2 * ps.min_piece)
    return 0;
  const int64_t by_work =
      items * ((max_work + ps.min_piece - 1) / ps.min_piece);
  return by_work < ps.max_parts() ? by_work : ps.max_parts();
}

// Estimated time of a cut, in blocks of a workgroup: the pieces run longest
// first on `slots` workgroups, so the launch takes its total divided by the
// slots plus what the last round leaves idle (as long as the shortest
// pieces), and never less than its longest piece; then the fold.
// parts < 0 if the cut needs more partials than there are.
struct Estimate {
  int64_t time, parts;
};
inline Estimate estimate(const int32_t* w, int32_t n, int32_t heads,
                         const Cut& s, const Pass& ps) {
  int64_t pieces = 0, parts = 0, sum = 0;
  int32_t longest = 0, shortest = INT32_MAX;
  for (int32_t i = 0; i < n; ++i) {
    const int32_t k = num_pieces(s, i, w[i]);
    pieces += k;
    if (k > 1) parts += k;
    sum += w[i];
    const int32_t hi = (w[i] + k - 1) / k, lo = w[i] / k;
    if (hi > longest) longest = hi;
    if (lo < shortest) shortest = lo;
  }
  pieces *= heads;
  parts *= heads;
  sum = sum * heads + pieces * ps.overhead;
  if (parts > ps.max_parts()) return {0, -1};
  const int64_t idle = (ps.slots - pieces % ps.slots) % ps.slots;
  int64_t t =
      (sum + idle * (shortest + ps.overhead) + ps.slots - 1) / ps.slots;
  if (t < longest + ps.overhead) t = longest + ps.overhead;
  return {t + (parts > 0 ? ps.fold + parts / ps.fold_rate : 0), parts};
}

// The cut of a tile for ps.slots, Cut{} to leave every item whole: the best
// estimate over the pieces of the longest item, and for equal items also whole
// rounds with only the rows of the last, partly filled round cut.  A cut has to
// be estimated 5 % faster than whole items.
inline Cut choose_alone(const int32_t* w, int32_t n, int32_t heads,
                  const Pass& ps) {
  const int64_t items = int64_t{n} * heads;
  int32_t longest = 0, shortest = INT32_MAX;
  for (int32_t i = 0; i < n; ++i) {
    if (w[i] > longest) longest = w[i];
    if (w[i] < shortest) shortest = w[i];
  }
  if (items > ps.max_items || longest <= 2 * ps.min_piece)
    return {};
  int64_t whole_time = estimate(w, n, heads, Cut{}, ps).time;
  if (ps.alone > 0 && 2 * items <= ps.slots) {
    const int64_t alone =
        (int64_t{longest} * ps.alone + 99) / 100 + ps.alone_overhead;
    if (alone < whole_time) whole_time = alone;
  }
  Cut best;
  int64_t best_time = whole_time * 19 / 20;
  auto consider = [&](const Cut& s) {
    const Estimate e = estimate(w, n, heads, s, ps);
    if (e.parts > 0 && e.time < best_time) {
      best_time = e.time;
      best = s;
    }
    return e.parts >= 0;
  };
  int32_t last = longest;
  for (int32_t k = 2;; ++k) {
    const int32_t c = (longest + k - 1) / k;
    if (c < ps.min_piece) break;
    if (c == last) continue;
    last = c;
    if (!consider({c, 0, ps.slots})) break;
  }
  if (longest == shortest && items > ps.slots) {
    const int32_t rounds = static_cast<int32_t>(items / ps.slots);
    const int32_t whole = rounds * ps.slots / heads;  // rows
    if (whole > 0 && whole < n) {
      const int64_t rest = items - int64_t{whole} * heads;
      const int64_t k =
          (int64_t{rounds + 1} * ps.slots - int64_t{whole} * heads) / rest;
      const int32_t c = static_cast<int32_t>((longest + k - 1) / k);
      if (k > 1 && c >= ps.min_piece) consider({c, whole, ps.slots});
    }
  }
  return best;
}

inline Cut choose(const int32_t* w, int32_t n, int32_t heads,
                  const Pass& ps) {
  const Cut best = choose_alone(w, n, heads, ps);
  return best.c == 0 && ps.beside ? choose_alone(w, n, heads, *ps.beside)
                                  : best;
}

}  // namespace split

// gfx950 (MI355X) has 8 XCDs; consecutive workgroup ids are dispatched to
// XCDs round robin, so id i runs on XCD i % 8.
constexpr int kNumXcd = 8;

// How the slots of a launch map to the pieces of one head, ranked, times the
// heads.  Plain: rank by rank, the heads of equal ranks together.  By KV
// head: XCD x (slots j * 8 + x) gets the pieces of KV heads x, x + 8, .., so
// that they share K and V in its L2 (KV heads a multiple of 8).  One round
// (a split tile of no more pieces than run at once, ranked by piece index):
// consecutive pieces of a KV head, which walk the same keys, share an XCD.
enum { kModePlain = 0, kModeByKv = 1, kModeOneRound = 2 };

__host__ __device__ inline int split_mode(int64_t total, bool is_split,
                                          bool by_kv, int32_t slots) {
  if (is_split && total <= slots) return kModeOneRound;
  return by_kv ? kModeByKv : kModePlain;
}

// Place of a slot: the KV-head and rank group it falls into.  A first look at
// entry `probe` of the ranked table gives its class, the entries [before,
// before + same) of equal rank; place_in_class then gives entry and head.
struct SlotPlace {
  int32_t probe;  // table entry whose class holds the slot
  int32_t at;     // position within the heads that share the class's line
  int32_t base;   // first KV head of that line
};

// m table entries, `heads` heads, `group` heads per KV head; slot < m * heads.
__host__ __device__ inline SlotPlace place_slot(int mode, int slot, int m,
                                                int heads, int group) {
  if (mode == kModePlain) return {slot / heads, slot, 0};
  const int x = slot % kNumXcd, j = slot / kNumXcd;
  if (mode == kModeByKv) return {j / (heads / kNumXcd), j, x};
  const int total = m * heads;
  const int len = total / kNumXcd, more = total % kNumXcd;
  const int pos = x < more ? x * (len + 1) + j : more + x * len + j;
  const int kvh = pos / (group * m), at = pos - kvh * group * m;
  return {at / group, at, kvh};
}

// Entry and head of the slot, given its class.
__host__ __device__ inline void place_in_class(int mode, const SlotPlace& s,
                                               int before, int same, int heads,
                                               int group, int* entry,
                                               int* head) {
  const int line = mode == kModePlain  ? heads
                   : mode == kModeByKv ? heads / kNumXcd
                                       : group;
  const int q = s.at - before * line;
  const int hl = q / same;  // head within the line
  *entry = before + q % same;
  *head = mode == kModePlain ? hl
          : mode == kModeByKv
              ? (hl / group * kNumXcd + s.base) * group + hl % group
              : s.base * group + hl;
}

}  // namespace mesh_attn
