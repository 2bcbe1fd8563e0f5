// CPU check of the classes of equal work items (csrc/class_plan.h): over seeded
// shapes of the forward and both kinds of the backward, the classes are those of a
// chunk-by-chunk walk, and calls of millions of chunks evaluate few costs.
#include "bwd_plan.h"
#include "fwd_plan.h"

#include <cstdio>
#include <cstdlib>
#include <random>
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

// The classes from a walk over all chunks: runs of equal ones, and where those are
// more than room - 1, groups of ceil(body / (room - 1)) chunks (at least 2).
template <typename Cost>
static std::vector<WorkClass> walk(int64_t n, int64_t per, int64_t per_last, int kind, int room, Cost cost) {
  const int64_t body = n - 1;
  std::vector<WorkClass> v;
  for (int64_t step = 1;; step = std::max<int64_t>(2 * step, cdiv(body, room - 1))) {
    v.clear();
    for (int64_t c = 0; c < body; c += step) {
      const int64_t nc = std::min(step, body - c);
      const int64_t w = std::max(std::max(cost(c), cost(c + nc - 1)), cost(c + nc / 2));
      if (!v.empty() && v.back().cost == w) {
        v.back().nc += (int32_t)nc;
        v.back().units += nc * per;
      } else {
        v.push_back(WorkClass{w, nc * per, (int32_t)c, (int32_t)nc, kind});
      }
    }
    if ((int64_t)v.size() <= room - 1) break;
  }
  v.push_back(WorkClass{cost(n - 1), per_last, (int32_t)(n - 1), 1, kind});
  return v;
}

// Checks the classes of one kind (0: forward, 1: dQ, 2: dK/dV); returns how many costs were evaluated.
static int64_t check(int64_t nq, int64_t nkv, int64_t L, int64_t off, int64_t W, int what, bool compare) {
  const int64_t nqc = cdiv(nq, L), nkc = cdiv(nkv, L);
  const ItemShape f{1, nqc, 1, 1, L, off, W, nkv, 96};
  const BwdShape b{1, nqc, 1, 1, nkc, 1, 1, L, off, W, nq, nkv};
  int64_t evals = 0;
  auto cost = [&](int64_t c) {
    ++evals;
    return what == 0 ? fwd_cost(chunk_key_tiles(f, c), false, 128)
                     : (what == 1 ? bwd_q_cost(bwd_q_tiles(b, c), 1) : bwd_kv_cost(bwd_kv_tiles(b, c), 1));
  };
  const int64_t n = what == 2 ? nkc : nqc;
  const int room = what == 0 ? kMaxClasses : kMaxClasses / 2;
  WorkClass cls[kMaxClasses];
  const int m = make_classes(n, 3, 2, what == 2, room, what == 2 ? off : n, cls, cost);
  const int64_t used = evals;
  CHECK(m >= 1 && m <= room);
  if (compare) {
    const std::vector<WorkClass> ref = walk(n, 3, 2, what == 2, room, cost);
    CHECK((int)ref.size() == m);
    for (int k = 0; k < m; ++k)
      CHECK(cls[k].cost == ref[k].cost && cls[k].units == ref[k].units && cls[k].c0 == ref[k].c0 &&
            cls[k].nc == ref[k].nc && cls[k].kind == ref[k].kind);
  }
  return used;
}

int main() {
  std::mt19937_64 rng(5);
  auto pick = [&](int64_t lo, int64_t hi) { return lo + (int64_t)(rng() % (uint64_t)(hi - lo + 1)); };
  int cases = 0;
  for (; cases < 3000; ++cases) {
    const int64_t L = pick(1, cases % 3 ? 12 : 300), nkv = pick(L, L * pick(1, 700));
    const int64_t off = pick(0, (nkv - 1) / L) / pick(1, 4), W = cases % 4 ? pick(0, cases % 5 ? 6 : 400) : -1;
    const int64_t nq = pick(1, nkv - off * L);
    for (int what = 0; what < 3; ++what) check(nq, nkv, L, off, W, what, true);
  }
  // one token a chunk, millions of chunks: windows, an unbounded prefix, a late query chunk
  for (int64_t n : {int64_t(65280), int64_t(4) << 20})
    for (int64_t W : {0, 1, 2, 40, 5000, -1})
      for (int64_t off : {int64_t(0), n / 2})
        for (int what = 0; what < 3; ++what, ++cases) CHECK(check(n - off, n, 1, off, W, what, false) < 1500);
  std::printf("%d cases ok\n", cases);
  return 0;
}
