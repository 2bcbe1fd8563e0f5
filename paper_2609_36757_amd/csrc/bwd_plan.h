// Work plan of the backward's gradient kernel (host code, plain C++).
//
// The kernel runs two kinds of work units in one launch, dQ units (a 256-row
// query tile against the keys it sees) and dK/dV units (a 128-key block against
// the queries that see it).  The plan groups the units into classes of equal
// length (one kind, a run of chunks) and orders the classes longest first:
// dispatch in that order is longest-first list scheduling over both kinds.
//
// With few units per CU it can pay to cut every unit of a kind in two along its
// summed axis (keys for dQ, queries for dK/dV).  The two halves add their sums
// into a zeroed output with one atomic add each: 0 + a + b is the same number
// in both orders, so the result stays reproducible bit for bit, which three or
// more parts would not be.  A simulated list schedule of the four choices
// decides.
#pragma once

#include <stdint.h>

#include <algorithm>

#include "class_plan.h"

namespace fastvr {

// Passed by value as a kernel argument.
struct BwdPlan {
  ClassTable tab;             // kind 0: dQ units, 1: dK/dV units
  int32_t q_split, kv_split;  // parts per unit (1 or 2)
};

// The call's decomposition (see FwdGrid / BwdGrid).
struct BwdShape {
  int64_t bh;
  int64_t n_qchunks, tiles_full, tiles_last;       // query chunks, 256-row tiles of one
  int64_t n_kchunks, kblocks_full, kblocks_last;   // key chunks, 128-key blocks of one
  int64_t chunk_len, q_chunk_offset, window, nq, nkv;  // window -1: unbounded
};

constexpr int64_t kBwdTile = 64;  // rows of a streamed tile

// Streamed tiles of a dQ unit of local query chunk c, and of a dK/dV unit of key chunk c.
inline int64_t bwd_q_tiles(const BwdShape& s, int64_t c) {
  const int64_t cg = s.q_chunk_offset + c, L = s.chunk_len;
  const int64_t lo = (s.window >= 0 && cg > s.window) ? (cg - s.window) * L : 0;
  const int64_t hi = (L < s.nkv - cg * L) ? (cg + 1) * L : s.nkv;
  return (hi - lo + kBwdTile - 1) / kBwdTile;
}
inline int64_t bwd_kv_tiles(const BwdShape& s, int64_t c) {
  const int64_t lo = std::max<int64_t>(c - s.q_chunk_offset, 0);
  int64_t hi = s.n_qchunks;
  if (s.window >= 0) hi = std::min(hi, c + s.window - s.q_chunk_offset + 1);
  if (hi <= lo) return 0;
  const int64_t qlo = lo * s.chunk_len, qhi = std::min(hi * s.chunk_len, s.nq);
  return qhi > qlo ? (qhi - qlo + kBwdTile - 1) / kBwdTile : 0;
}

// Narrows rows lo .. hi - 1, the summed axis of a unit cut in two, to part `half`:
// whole tiles, the first part the longer.  False if nothing is left.  (The kernel
// calls it too: a constexpr function is compiled for host and device.)
constexpr bool bwd_half_rows(int half, int& lo, int& hi) {
  constexpr int kTile = (int)kBwdTile;
  const int mid = lo + ((hi - lo + kTile - 1) / kTile + 1) / 2 * kTile;
  if (half == 0)
    hi = mid < hi ? mid : hi;
  else
    lo = mid;
  return lo < hi;
}

// Unit costs in thirds of a dK/dV tile (about 0.6 us).  Fitted to the times of
// the four split choices on eleven shapes (head_dim 64 and 128, 24 to 900
// units; 4 to 5% rms): a dQ tile counts 4/3 of a dK/dV tile, a unit's prologue and
// epilogue 6 tiles, and 10 when it adds its sums to a zeroed output; the adds of
// all units (2 TB/s, against 4.9 TB/s of a copy) take 2 tiles a unit and CU more.
constexpr int64_t kBwdUnitCost = 18, kBwdSplitUnitCost = 30, kBwdSplitAddCost = 6;
inline int64_t bwd_q_cost(int64_t tiles, int64_t split) {
  return 4 * ((tiles + split - 1) / split) + (split > 1 ? kBwdSplitUnitCost : kBwdUnitCost);
}
inline int64_t bwd_kv_cost(int64_t tiles, int64_t split) {
  return 3 * ((tiles + split - 1) / split) + (split > 1 ? kBwdSplitUnitCost : kBwdUnitCost);
}

// The classes of one kind in chunk order.
inline int bwd_classes(const BwdShape& s, bool kv, int64_t split, WorkClass* out) {
  const int64_t n = kv ? s.n_kchunks : s.n_qchunks;
  const int64_t per = (kv ? s.kblocks_full : s.tiles_full) * s.bh * split;
  const int64_t per_last = (kv ? s.kblocks_last : s.tiles_last) * s.bh * split;
  // a query chunk sees more keys the later it is, up to the window; a key chunk is
  // seen by more queries up to the first query chunk, and by fewer after it
  const int64_t peak = kv ? s.q_chunk_offset : n;
  return make_classes(n, per, per_last, kv ? 1 : 0, kMaxClasses / 2, peak, out, [&](int64_t c) {
    return kv ? bwd_kv_cost(bwd_kv_tiles(s, c), split) : bwd_q_cost(bwd_q_tiles(s, c), split);
  });
}

// Both kinds' classes, longest first.
inline int bwd_sorted_classes(const BwdShape& s, int64_t q_split, int64_t kv_split, WorkClass* out) {
  int n = bwd_classes(s, true, kv_split, out);
  n += bwd_classes(s, false, q_split, out + n);
  sort_classes(out, n);
  return n;
}

// Units per CU up to which the split choices are simulated.  At 3.5 (9 chunks of
// 1333, 8 heads) the best split was already 1% slower than none; at 1.5 (2 heads,
// 8000 keys) and below splits gained 5 to 40%.
constexpr int64_t kBwdSplitMaxRounds = 4;

// Fills the plan; returns the number of units (the grid).  may_split: the outputs
// lie in memory that the halves' atomic adds are defined on.
inline int64_t bwd_plan(const BwdShape& s, int n_cu, bool may_split, BwdPlan* p) {
  WorkClass cls[kMaxClasses], best[kMaxClasses];
  int n = bwd_sorted_classes(s, 1, 1, best);
  p->q_split = p->kv_split = 1;
  int64_t units = 0;
  for (int k = 0; k < n; ++k) units += best[k].units;
  if (may_split && n_cu > 0 && n_cu <= 256 && units <= kBwdSplitMaxRounds * n_cu) {
    int64_t span = class_makespan(best, n, n_cu);
    for (int opt = 1; opt < 4; ++opt) {
      const int m = bwd_sorted_classes(s, (opt & 1) ? 2 : 1, (opt & 2) ? 2 : 1, cls);
      int64_t added = 0;
      for (int k = 0; k < m; ++k) added += (opt & (cls[k].kind ? 2 : 1)) ? cls[k].units : 0;
      const int64_t t = class_makespan(cls, m, n_cu) + kBwdSplitAddCost * added / n_cu;
      if (25 * t < 24 * span) {  // 4% at least: the model is no better than that
        span = t;
        n = m;
        std::copy(cls, cls + m, best);
        p->q_split = (opt & 1) ? 2 : 1;
        p->kv_split = (opt & 2) ? 2 : 1;
      }
    }
  }
  return fill_table(best, n, &p->tab);
}

}  // namespace fastvr
