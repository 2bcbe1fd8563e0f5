// Work plan of the forward's plain dispatch (host code, plain C++): the class
// table, and whether the call runs 128-row or 256-row items.
//
// A 256-row item keeps both waves of every SIMD at matrix-core and softmax work
// in turn and has the higher throughput.  A 128-row item, whose SIMD pair shares
// 32 rows, ends sooner: 1.28 against 2.05 us a key tile (head_dim 128), 0.77
// against 1.58 us (head_dim 64), but at full load two of them take 1.14 (1.11)
// times a 256-row item's time.  So the plan simulates the list schedule of both
// and takes 128-row items where their schedule ends at least 4% sooner: calls
// that leave CUs idle, or whose last wave of 256-row items is nearly empty.
#pragma once

#include <stdint.h>

#include "class_plan.h"
#include "item_lists.h"

namespace fastvr {

constexpr int kHalfRows = 128;

struct FwdPlan {
  ClassTable tab;
  bool half;
};

// Items per CU up to which 128-row items are considered.
constexpr int64_t kHalfMaxRounds = 4;

// Item costs in 1/25 of a 256-row item's key tile, three tiles for prologue and
// epilogue: a 128-row item's key tile counts 16/25 (head_dim 128) or 14/25 (64).
inline int64_t fwd_cost(int64_t key_tiles, bool half, int d) {
  return (half ? (d == 128 ? 16 : 14) : 25) * key_tiles + 75;
}

// s: the call with its 256-row tiles; half_full / half_last: 128-row tiles of a
// full and of the last chunk.
inline void fwd_plan(const ItemShape& s, int64_t half_full, int64_t half_last, int d, int n_cu, FwdPlan* p) {
  auto classes = [&](bool half, WorkClass* out) {
    const int64_t per = s.bh * (half ? half_full : s.tiles_full), last = s.bh * (half ? half_last : s.tiles_last);
    const int n = make_classes(s.n_local_chunks, per, last, 0, kMaxClasses, out,
                               [&](int64_t c) { return fwd_cost(chunk_key_tiles(s, c), half, d); });
    sort_classes(out, n);
    return n;
  };
  WorkClass full[kMaxClasses], half[kMaxClasses];
  const int n = classes(false, full);
  int64_t units = 0;
  for (int k = 0; k < n; ++k) units += full[k].units;
  p->half = false;
  if (n_cu > 0 && n_cu <= 256 && units <= kHalfMaxRounds * n_cu) {
    const int m = classes(true, half);
    if (25 * class_makespan(half, m, n_cu) < 24 * class_makespan(full, n, n_cu)) {
      p->half = true;
      fill_table(half, m, &p->tab);
      return;
    }
  }
  fill_table(full, n, &p->tab);
}

}  // namespace fastvr
