// CPU check of the forward's work plan (csrc/fwd_plan.h): over seeded shapes every
// (chunk, batch * head, tile) comes from exactly one item index with either item
// height, and the heights chosen for a few shapes.
#include "fwd_plan.h"

#include <cstdio>
#include <cstdlib>
#include <random>
#include <set>
#include <tuple>

using namespace fastvr;

#define CHECK(x)                                         \
  do {                                                   \
    if (!(x)) {                                          \
      std::printf("line %d: %s failed\n", __LINE__, #x); \
      std::exit(1);                                      \
    }                                                    \
  } while (0)

static int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Rows of the call's items.
static int check(int64_t bh, int64_t nq, int64_t nkv, int64_t L, int64_t off, int64_t W, int d, int n_cu = 256) {
  if (L > nkv) L = nkv;
  const int64_t nc = cdiv(nq, L), last = nq - (nc - 1) * L;
  ItemShape s{bh, nc, nc > 1 ? cdiv(L, 256) : cdiv(last, 256), cdiv(last, 256), L, off, W, nkv, 96};
  FwdPlan p;
  fwd_plan(s, last, d, n_cu, &p);
  const int64_t hl = cdiv(last, p.rows), hf = nc > 1 ? cdiv(L, p.rows) : hl;
  CHECK(p.half == (p.rows == 128) && p.rows % 32 == 0 && p.tiles_full == hf && p.tiles_last == hl);
  std::set<std::tuple<int64_t, int64_t, int64_t>> seen;
  for (int k = 0; k < p.tab.n; ++k)
    for (int i = 0; i < p.tab.first[k + 1] - p.tab.first[k]; ++i) {
      const int64_t u = xcd_unit(i, p.tab.first[k + 1] - p.tab.first[k]);
      const int64_t t = p.tab.c0[k] == nc - 1 ? hl : hf, c = p.tab.c0[k] + u / (bh * t);
      CHECK(c < p.tab.c0[k] + p.tab.nc[k] && c < nc);
      CHECK(seen.insert({c, u % (bh * t) / t, u % t}).second);
    }
  CHECK((int64_t)seen.size() == bh * (hl + hf * (nc - 1)));
  if (p.rows != 256 && p.rows != 128) CHECK((int64_t)seen.size() <= n_cu);
  return p.rows;
}

int main() {
  std::mt19937_64 rng(11);
  auto pick = [&](int64_t lo, int64_t hi) { return lo + (int64_t)(rng() % (uint64_t)(hi - lo + 1)); };
  int n = 0, halves = 0, low = 0;
  for (; n < 400; ++n) {
    const int64_t nkv = pick(1, 4000), L = pick(1, 900), off = std::min<int64_t>(pick(0, 3), (nkv - 1) / std::min(L, nkv));
    const int rows = check(pick(1, 24), pick(1, nkv - off * std::min(L, nkv)), nkv, L, L > nkv ? 0 : off, pick(-1, 4),
                           n % 2 ? 64 : 128, n % 3 ? 256 : (int)pick(1, 256));
    halves += rows == 128;
    low += rows > 128 && rows < 256;
  }
  CHECK(halves > 40 && halves < 360 && low > 5);
  // 8 and 128 items of 256 rows leave CUs idle; 156 would need two waves of 128-row
  // items, but 240 of 160 rows still run at once; 768 fill the chip
  CHECK(check(2, 1024, 1024, 256, 0, -1, 64) == 128 && check(4, 8192, 8192, 8192, 0, -1, 128) == 128);
  CHECK(check(12, 3120, 12480, 3120, 3, -1, 128) == 160 && check(12, 16320, 65280, 16320, 3, -1, 128) == 256);
  // the shapes of tests/test_gpu_half_items.py
  for (int d = 64; d <= 128; d += 64) {
    CHECK(check(2, 900, 900, 259, 0, -1, d) == 128 && check(2, 259, 518, 259, 1, 1, d) == 128);
    CHECK(check(256, 900, 900, 259, 0, -1, d) == 256 && check(512, 259, 518, 259, 1, 1, d) == 256);
    CHECK(check(80, 650, 1300, 650, 1, -1, d) == 224 && check(62, 650, 1300, 650, 1, -1, d) == 192);
    CHECK(check(50, 650, 1300, 650, 1, -1, d) == 160);
    // its ring steps: chunk 3 with chunk 2 in the ring
    const int64_t L = d == 128 ? 260 : 264;
    CHECK(check(2, 200, L + 200, L, 1, 1, d) == 128 && check(512, 200, L + 200, L, 1, 1, d) == 256);
    CHECK(check(80, 650, 1306, 656, 1, 1, d) == 224 && check(62, 650, 1306, 656, 1, 1, d) == 192);
    CHECK(check(50, 650, 1306, 656, 1, 1, d) == 160 && check(512, 650, 1306, 656, 1, 1, d) == 256);
  }
  // the far streaming chunk of tests/test_gpu_full_items.py: one 256-row item per CU
  CHECK(check(2, 32768, 258 * 32768, 32768, 257, 1, 128) == 256);
  // more than four 256-row items per CU (tests/test_gpu_full_items.py: over 1024 heads)
  for (int i = 0; i < 60; ++i, ++n) {
    const int64_t nkv = pick(1, 1500), L = pick(1, 900), off = std::min<int64_t>(pick(0, 3), (nkv - 1) / std::min(L, nkv));
    CHECK(check(pick(1025, 1028), pick(1, nkv - off * std::min(L, nkv)), nkv, L, L > nkv ? 0 : off, pick(-1, 4),
                i % 2 ? 64 : 128) == 256);
  }
  std::printf("%d cases ok\n", n);
  return 0;
}
