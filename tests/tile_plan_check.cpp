// CPU check of the tile gather's launch plan (csrc/tile_plan.h): over seeded
// geometries, the workgroups and threads of the launch write every (tile, row,
// unit) exactly once, from the field unit it is a copy of; calls with few rows and
// many tiles per position are spread over workgroups, rows of few units over waves.
#include "tile_plan.h"

#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

using namespace fastvr;

#define CHECK(x)                                         \
  do {                                                   \
    if (!(x)) {                                          \
      std::printf("line %d: %s failed\n", __LINE__, #x); \
      std::exit(1);                                      \
    }                                                    \
  } while (0)

static Axis axis(int size, int tile, int overlap) {
  const int L = std::min(size, tile);
  const int n = size <= tile ? 1 : (size - overlap + (tile - overlap) - 1) / (tile - overlap);
  return Axis{n, L, size - L};
}

// The kernel's loops over one launch, thread by thread.
template <typename I>
static GatherGrid check(int frames, int Hg, int Wg, int C16, int tile, int overlap) {
  const Axis ay = axis(Hg, tile, overlap), ax = axis(Wg, tile, overlap);
  const int64_t rows = (int64_t)frames * Hg;
  const GatherGrid g = gather_grid(rows, Wg, C16, ay, ax);
  CHECK((g.width == 64 || g.width == kTileThreads) && g.seg <= g.width * kGatherUnits && g.seg >= 1);
  CHECK(g.segments >= 1 && g.segments * g.seg >= (int64_t)Wg * C16 && (g.segments - 1) * g.seg < (int64_t)Wg * C16);
  CHECK(g.row_groups >= 1 && g.row_groups <= 65535 && g.zy >= 1 && g.zx >= 1 && g.zy * g.zx <= 65535);
  const int row_units = Wg * C16, tile_units = ax.L * C16, per = kTileThreads / g.width;
  std::vector<int> src((int64_t)frames * ay.n * ax.n * ay.L * tile_units, -1);
  for (int z = 0; z < g.zy * g.zx; ++z)
    for (int64_t by = 0; by < g.row_groups; ++by)
      for (int64_t bx = 0; bx < g.segments; ++bx) {
        const int u_begin = (int)bx * g.seg, u_end = std::min(u_begin + g.seg, row_units);
        const int tx_hi = last_start_le<I>(ax, (u_end - 1) / C16);
        const int ty_part = z % g.zy, tx_lo = first_end_gt<I>(ax, u_begin / C16) + z / g.zy;
        for (int sub = 0; sub < per; ++sub)
          for (int64_t r = by * per + sub; r < rows; r += g.row_groups * per) {
            const int y = (int)(r % Hg), f = (int)(r / Hg);
            for (int ty = first_end_gt<I>(ay, y) + ty_part; ty <= last_start_le<I>(ay, y); ty += g.zy)
              for (int tx = tx_lo; tx <= tx_hi; tx += g.zx) {
                const int u0 = origin_t<I>(ax, tx) * C16, iy = y - origin_t<I>(ay, ty);
                CHECK(ty < ay.n && tx < ax.n && iy >= 0 && iy < ay.L);
                const int64_t row = ((int64_t)(ty * ax.n + tx) * frames + f) * ay.L + iy;
                for (int u = u_begin; u < u_end; ++u) {  // threads and their units
                  const int v = u - u0;
                  if (v < 0 || v >= tile_units) continue;
                  int& s = src[row * tile_units + v];
                  CHECK(s == -1);
                  s = (int)(r * row_units + u);
                }
              }
          }
      }
  for (int ty = 0; ty < ay.n; ++ty)
    for (int tx = 0; tx < ax.n; ++tx)
      for (int f = 0; f < frames; ++f)
        for (int iy = 0; iy < ay.L; ++iy)
          for (int v = 0; v < tile_units; ++v) {
            const int64_t row = ((int64_t)(ty * ax.n + tx) * frames + f) * ay.L + iy;
            const int want = (f * Hg + origin_t<I>(ay, ty) + iy) * row_units + origin_t<I>(ax, tx) * C16 + v;
            CHECK(src[row * tile_units + v] == want);
          }
  return g;
}

int main() {
  std::mt19937_64 rng(3);
  auto pick = [&](int lo, int hi) { return lo + (int)(rng() % (uint64_t)(hi - lo + 1)); };
  int cases = 0, waves = 0, shared = 0;
  while (cases < 400) {
    const int frames = pick(1, 3), Hg = pick(1, 60), Wg = pick(1, 60), C16 = pick(1, pick(1, 60)), tile = pick(1, 40);
    const int overlap = pick(cases % 3 ? 0 : tile - 1 - tile / 8, tile - 1);
    const Axis ay = axis(Hg, tile, overlap), ax = axis(Wg, tile, overlap);
    if ((int64_t)frames * ay.n * ax.n * ay.L * ax.L * C16 > 3000000) continue;
    const GatherGrid g = cases % 2 ? check<uint32_t>(frames, Hg, Wg, C16, tile, overlap)
                                   : check<uint64_t>(frames, Hg, Wg, C16, tile, overlap);
    waves += g.width == 64;
    shared += g.zy * g.zx > 1;
    ++cases;
  }
  std::printf("%d by waves, %d shared\n", waves, shared);
  CHECK(waves > 100 && waves < 380 && shared > 40 && shared < 360);
  // fields of a few units a row: a wave per row
  CHECK(gather_grid(64 * 8 * 30, 30, 2, axis(30, 64, 16), axis(30, 64, 16)).width == 64);
  // 768 + 32 units would be an uneven pair of segments
  CHECK(gather_grid(4096, 100, 8, axis(64, 64, 16), axis(100, 64, 16)).seg == 448);
  // 100 rows, 1369 tiles: spread; 544 rows of 30 segments with 6 tiles: one workgroup per place
  const GatherGrid many = gather_grid(100, 100, 6, axis(100, 64, 63), axis(100, 64, 63));
  CHECK(many.segments * many.row_groups * many.zy * many.zx >= kGatherBlocks / 2);
  const GatherGrid few = gather_grid(8 * 68, 120, 192, axis(68, 64, 16), axis(120, 64, 16));
  CHECK(few.zy * few.zx == 1 && few.width == kTileThreads && few.segments == 30 && few.seg == 768);
  // shapes of tests/test_gpu_tile_paths.py
  const GatherGrid a = gather_grid(6 * 40, 45, 48, axis(40, 32, 30), axis(45, 32, 30));
  const GatherGrid b = gather_grid(6 * 40, 45, 5, axis(40, 32, 31), axis(45, 32, 31));
  CHECK(a.width == kTileThreads && a.zy * a.zx > 1 && b.width == 64 && b.zy * b.zx > 1);
  std::printf("%d cases ok\n", cases);
  return 0;
}
