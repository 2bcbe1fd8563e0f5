// CPU check of the backward's work plan (csrc/bwd_plan.h): over seeded shapes,
// every (kind, chunk, batch * head, block, half) is decoded from exactly one
// unit index, the halves of a split unit hold every streamed tile once, classes
// are ordered longest first, and the grouped makespan equals a plain simulation.
#include "bwd_plan.h"

#include <cstdio>
#include <cstdlib>
#include <random>
#include <set>
#include <tuple>
#include <vector>

using namespace fastvr;

#define CHECK(x)                                              \
  do {                                                        \
    if (!(x)) {                                               \
      std::printf("line %d: %s failed\n", __LINE__, #x);      \
      std::exit(1);                                           \
    }                                                         \
  } while (0)

static int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

static BwdShape make(int64_t bh, int64_t nq, int64_t nkv, int64_t L, int64_t off, int64_t W) {
  if (L > nkv) L = nkv;
  BwdShape s{};
  s.bh = bh;
  s.n_qchunks = nq > 0 ? cdiv(nq, L) : 0;
  if (nq > 0) {
    s.tiles_last = cdiv(nq - (s.n_qchunks - 1) * L, 256);
    s.tiles_full = s.n_qchunks > 1 ? cdiv(L, 256) : s.tiles_last;
  }
  s.n_kchunks = cdiv(nkv, L);
  s.kblocks_last = cdiv(nkv - (s.n_kchunks - 1) * L, 128);
  s.kblocks_full = s.n_kchunks > 1 ? cdiv(L, 128) : s.kblocks_last;
  s.chunk_len = L;
  s.q_chunk_offset = off;
  s.window = W;
  s.nq = nq;
  s.nkv = nkv;
  return s;
}

static void check(const BwdShape& s, int n_cu) {
  BwdPlan p;
  const int64_t n = bwd_plan(s, n_cu, true, &p);
  CHECK(p.tab.n >= 1 && p.tab.n <= kMaxClasses && p.tab.first[0] == 0 && p.tab.first[p.tab.n] == n);
  CHECK((p.q_split == 1 || p.q_split == 2) && (p.kv_split == 1 || p.kv_split == 2));
  std::set<std::tuple<int, int64_t, int64_t, int64_t, int64_t>> seen;
  // the table is the sorted classes, by the cost they were sorted by
  WorkClass cls[kMaxClasses];
  CHECK(bwd_sorted_classes(s, p.q_split, p.kv_split, cls) == p.tab.n);
  int64_t prev = INT64_MAX;
  for (int k = 0; k < p.tab.n; ++k) {
    CHECK(cls[k].cost <= prev && cls[k].c0 == p.tab.c0[k] && cls[k].nc == p.tab.nc[k] && cls[k].kind == p.tab.kind[k]);
    prev = cls[k].cost;
    const bool kv = p.tab.kind[k] != 0;
    const int64_t split = kv ? p.kv_split : p.q_split, last = (kv ? s.n_kchunks : s.n_qchunks) - 1;
    const int64_t blocks = kv ? (p.tab.c0[k] == last ? s.kblocks_last : s.kblocks_full)
                              : (p.tab.c0[k] == last ? s.tiles_last : s.tiles_full);
    int64_t longest = 0;
    for (int64_t u = p.tab.first[k]; u < p.tab.first[k + 1]; ++u) {
      int64_t r = xcd_unit((int)(u - p.tab.first[k]), p.tab.first[k + 1] - p.tab.first[k]);
      const int64_t per_bh = blocks * split, per_c = per_bh * s.bh;
      const int64_t c = p.tab.c0[k] + r / per_c;
      CHECK(r / per_c < p.tab.nc[k]);
      r %= per_c;
      const int64_t bh = r / per_bh, t = r % per_bh / split, half = r % split;
      CHECK(c <= last && bh < s.bh && half < split);
      CHECK(seen.insert({kv ? 1 : 0, c, bh, half, t}).second);
      longest = std::max(longest, kv ? bwd_kv_cost(bwd_kv_tiles(s, c), split) : bwd_q_cost(bwd_q_tiles(s, c), split));
    }
    // a class of one run of equal chunks costs what each of its units does
    const int64_t n_runs_max = kMaxClasses / 2;
    if ((kv ? s.n_kchunks : s.n_qchunks) <= n_runs_max) CHECK(longest == cls[k].cost);
  }
  const int64_t q_units = s.n_qchunks ? s.bh * p.q_split * (s.tiles_last + s.tiles_full * (s.n_qchunks - 1)) : 0;
  const int64_t kv_units = s.bh * p.kv_split * (s.kblocks_last + s.kblocks_full * (s.n_kchunks - 1));
  CHECK(n == q_units + kv_units && (int64_t)seen.size() == n);
}

// The two parts of rows lo .. hi - 1: every row once, the first from lo in whole
// tiles unless it is alone, neither more than a tile longer than the other.
static void check_halves(int lo, int hi) {
  int a0 = lo, a1 = hi, b0 = lo, b1 = hi;
  const bool a = bwd_half_rows(0, a0, a1), b = bwd_half_rows(1, b0, b1);
  CHECK(a == (lo < hi) && b == (cdiv(hi - lo, kBwdTile) > 1));
  if (!a) return;
  CHECK(a0 == lo && a1 == (b ? b0 : hi));
  if (!b) return;
  CHECK(b1 == hi && (a1 - a0) % kBwdTile == 0);
  const int64_t ta = cdiv(a1 - a0, kBwdTile), tb = cdiv(b1 - b0, kBwdTile);
  CHECK(ta + tb == cdiv(hi - lo, kBwdTile) && (ta == tb || ta == tb + 1));
}

int main() {
  std::mt19937_64 rng(7);
  for (int lo : {0, 1, 63, 230, 5000})
    for (int n = 0; n <= 1200; ++n) check_halves(lo, lo + n);
  // the workgroup remap: a permutation, within each round of 256, for every class size
  for (int n = 1; n <= 1100; ++n) {
    std::vector<char> hit(n, 0);
    for (int i = 0; i < n; ++i) {
      const int u = xcd_unit(i, n);
      CHECK(u >= 0 && u < n && u / 256 == i / 256 && !hit[u]);
      hit[u] = 1;
    }
  }
  auto pick = [&](int64_t lo, int64_t hi) { return lo + (int64_t)(rng() % (uint64_t)(hi - lo + 1)); };
  int cases = 0;
  check(make(2, 1024, 1024, 256, 0, -1), 256), ++cases;
  check(make(12, 18720, 18720, 3120, 0, -1), 256), ++cases;
  check(make(2, 0, 300, 100, 0, -1), 256), ++cases;
  check(make(1, 1, 1, 5, 0, -1), 256), ++cases;
  check(make(2, 5000, 5000, 1, 0, 3), 256), ++cases;  // thousands of chunks
  for (int i = 0; i < 300; ++i) {
    const int64_t L = pick(1, 700), nkv = pick(1, 4000), W = pick(-1, 4);
    const int64_t off = std::min<int64_t>(pick(0, 3), (nkv - 1) / std::min(L, nkv));
    const int64_t room = nkv - off * std::min(L, nkv);
    check(make(pick(1, 24), pick(1, room), nkv, L, L > nkv ? 0 : off, W), i % 3 ? 256 : (int)pick(1, 256));
    ++cases;
  }
  // the splits that tests/test_gpu_bwd_split.py runs
  const BwdShape gpu[5] = {make(8, 1616, 1616, 230, 0, -1), make(2, 300, 900, 300, 2, -1), make(2, 1537, 1537, 500, 0, -1),
                           make(1, 2105, 2105, 100, 0, -1), make(1, 1300, 3900, 1300, 2, 0)};
  for (int i = 0; i < 5; ++i) {
    BwdPlan p;
    bwd_plan(gpu[i], 256, true, &p);
    CHECK(p.q_split == 2 && p.kv_split == (i < 2 ? 1 : 2));
    // outputs that take no atomic adds: no halves
    bwd_plan(gpu[i], 256, false, &p);
    CHECK(p.q_split == 1 && p.kv_split == 1);
  }
  // more than four units per CU (tests/test_gpu_full_items.py: over 1024 heads): whole units
  for (int i = 0; i < 40; ++i, ++cases) {
    const int64_t L = pick(1, 700), nkv = pick(1, 1500), off = std::min<int64_t>(pick(0, 3), (nkv - 1) / std::min(L, nkv));
    BwdPlan p;
    bwd_plan(make(pick(1025, 1028), pick(1, nkv - off * std::min(L, nkv)), nkv, L, L > nkv ? 0 : off, pick(-1, 4)), 256,
             true, &p);
    CHECK(p.q_split == 1 && p.kv_split == 1);
  }
  // the grouped schedule against CU-by-CU simulation
  for (int i = 0; i < 200; ++i, ++cases) {
    WorkClass cls[kMaxClasses];
    const int n = (int)pick(1, kMaxClasses), cu = (int)pick(1, 256);
    std::vector<int64_t> load(cu, 0);
    int64_t cost = pick(50, 400);
    for (int k = 0; k < n; ++k) {
      cls[k] = WorkClass{cost, pick(1, 300), 0, 1, 0};
      cost -= std::min(cost - 1, pick(0, 12));
      for (int64_t u = 0; u < cls[k].units; ++u) *std::min_element(load.begin(), load.end()) += cls[k].cost;
    }
    CHECK(class_makespan(cls, n, cu) == *std::max_element(load.begin(), load.end()));
  }
  std::printf("%d cases ok\n", cases);
  return 0;
}
