// Work plan of the forward's plain dispatch (host code, plain C++): the class
// table, and the height of the call's items.
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
  bool half;             // 128-row items (rows = 128)
  int32_t rows;          // query rows of an item
  int64_t tiles_full, tiles_last;  // items of a full and of the last chunk
};

// Heights of a call whose 256-row items all run at once, on no more than the
// CUs: the lowest that still does.  A CU's time falls a little with its rows
// (156 items of 256 rows 280 us; 204 of 192 rows 267; 240 of 160 rows 263; fewer
// waves at the LDS), and the CUs that had no item take the rest.  It falls no
// further because 160 rows are five 32-row waves on four SIMDs: the SIMD with two
// of them needs as long for a key tile as with 256 rows, and the others, with one
// wave each, leave their matrix cores idle in every second slot.
constexpr int kLowHeights[] = {160, 192, 224};

// Items per CU up to which 128-row items are considered.
constexpr int64_t kHalfMaxRounds = 4;

// Item costs in 1/25 of a 256-row item's key tile, three tiles for prologue and
// epilogue: a 128-row item's key tile counts 16/25 (head_dim 128) or 14/25 (64).
inline int64_t fwd_cost(int64_t key_tiles, bool half, int d) {
  return (half ? (d == 128 ? 16 : 14) : 25) * key_tiles + 75;
}

// s: the call with its 256-row tiles; last_rows: query rows of its last chunk.
inline void fwd_plan(const ItemShape& s, int64_t last_rows, int d, int n_cu, FwdPlan* p) {
  WorkClass cls[2][kMaxClasses];
  auto classes = [&](int rows, WorkClass* out) {
    const int64_t last = (last_rows + rows - 1) / rows;
    const int64_t full = s.n_local_chunks > 1 ? (s.chunk_len + rows - 1) / rows : last;
    p->half = rows == kHalfRows;
    p->rows = rows;
    p->tiles_full = full;
    p->tiles_last = last;
    const int n = make_classes(s.n_local_chunks, s.bh * full, s.bh * last, 0, kMaxClasses, s.n_local_chunks, out,
                               [&](int64_t c) { return fwd_cost(chunk_key_tiles(s, c), p->half, d); });
    sort_classes(out, n);
    return n;
  };
  auto items = [&]() { return s.bh * (p->tiles_last + p->tiles_full * (s.n_local_chunks - 1)); };
  int n = classes(256, cls[0]);
  const int64_t units = items();
  if (n_cu > 0 && n_cu <= 256 && units <= kHalfMaxRounds * n_cu) {
    const int64_t span = class_makespan(cls[0], n, n_cu);
    const int m = classes(kHalfRows, cls[1]);
    if (25 * class_makespan(cls[1], m, n_cu) < 24 * span) {
      fill_table(cls[1], m, &p->tab);
      return;
    }
    if (units <= n_cu)
      for (int rows : kLowHeights) {
        n = classes(rows, cls[0]);
        if (items() <= n_cu) {
          fill_table(cls[0], n, &p->tab);
          return;
        }
      }
    n = classes(256, cls[0]);
  }
  fill_table(cls[0], n, &p->tab);
}

}  // namespace fastvr
