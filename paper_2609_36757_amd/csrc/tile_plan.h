// Tiles along an axis, and the launch plan of the tile gather (plain C++; the
// constexpr functions are compiled for kernels and host alike).
#pragma once

#include <stdint.h>

#include <algorithm>

namespace fastvr {

constexpr int kTileThreads = 256;   // threads of a workgroup
constexpr int kGatherUnits = 3;     // 16-byte units of a field row that a thread holds

struct Axis {
  int n, L, span;  // tiles, tile length, size - L
};

// Index arithmetic in type I: uint32_t when every numerator below
// fits (the usual case), uint64_t otherwise.
template <typename I>
constexpr int origin_t(const Axis& a, int k) {
  return a.n == 1 ? 0 : (int)(((I)k * (I)a.span + (I)((a.n - 1) / 2)) / (I)(a.n - 1));
}

// Last tile starting at or before position p: the largest k with origin(k) <= p.
// origin(k) <= p  <=>  k * span + (n - 1) / 2 < (p + 1)(n - 1), solved for k.
template <typename I>
constexpr int last_start_le(const Axis& a, int p) {
  if (a.n == 1) return 0;
  const I num = (I)(p + 1) * (I)(a.n - 1) - (I)((a.n - 1) / 2) - 1;
  const I k = num / (I)a.span;  // span > 0 whenever n > 1
  return k < (I)(a.n - 1) ? (int)k : a.n - 1;
}

// First tile ending after position p: the smallest k with origin(k) + L > p,
// i.e. one past the last tile starting at or before p - L.
template <typename I>
constexpr int first_end_gt(const Axis& a, int p) {
  const int m = p - a.L;
  return m < 0 ? 0 : last_start_le<I>(a, m) + 1;
}

// The launch: workgroups of (width, kTileThreads / width) threads, `width` of them
// along a field row; grid (segments of seg units, row groups, zy * zx), where the zy *
// zx workgroups of one place share the tiles that cover it.
struct GatherGrid {
  int width, seg;
  int64_t segments, row_groups;
  int zy, zx;
};

// Tile rows of up to this many units: one wave per field row instead of the whole
// workgroup, whose four waves would have little of such a row each, or nothing.
// 64 x 8 fields of 30 x 30, 16 channels (60 units, one tile) 24.5 -> 9.1 us; 2 x
// 12 x 487 x 5, 152 channels (95 units) 23.7 -> 9.2; 2 x 10 x 344 x 61, 128
// channels, tiles of 19 (304 units) 44.4 -> 39.2.  At 384 units (100 x 100, 48
// channels, tiles of 64 one position apart) a wave per row took 155 and a workgroup 132 us.
constexpr int kGatherWaveUnits = 320;
// Workgroups that a call should have, and tiles of one place up to which one
// workgroup writes them all.  With fewer workgroups, as a small field cut into many
// overlapping tiles has, those of one place share its tiles: 300 x 300, 8 channels,
// tiles of 16 one position apart (256 per position) 811 -> 117 us; 130 x 130, 64
// channels, tiles of 64 four apart 52.0 -> 29.8.  Half as many workgroups took 6 to
// 12% more time on those two; parts of 8 tiles instead of 16 took 18 instead of 15 us
// on 2 x 8 x 470 x 33, 16 channels, tiles of 2, and no less anywhere.
constexpr int64_t kGatherBlocks = 4096, kGatherPartTiles = 16;

// Upper bound of the tiles that hold any of w consecutive positions.
inline int64_t tiles_over(const Axis& a, int64_t w) {
  return a.n == 1 ? 1 : std::min<int64_t>(a.n, (w + a.L - 2) * (a.n - 1) / a.span + 1);
}

inline GatherGrid gather_grid(int64_t rows, int64_t Wg, int64_t C16, const Axis& ay, const Axis& ax) {
  GatherGrid g;
  g.width = ax.L * C16 <= kGatherWaveUnits ? 64 : kTileThreads;
  // equal segments: workgroups alternate over the XCDs, so a short last one would
  // leave half of them with less work where a row has two
  const int64_t row_units = Wg * C16, per = kTileThreads / g.width;
  g.segments = (row_units + g.width * kGatherUnits - 1) / (g.width * kGatherUnits);
  g.seg = (int)(((row_units + g.segments - 1) / g.segments + 63) / 64 * 64);
  g.row_groups = std::min<int64_t>((rows + per - 1) / per, 65535);
  const int64_t ny = tiles_over(ay, 1), nx = tiles_over(ax, std::min(Wg, (g.seg + C16 - 2) / C16 + 1));
  const int64_t need = (kGatherBlocks + g.segments * g.row_groups - 1) / (g.segments * g.row_groups);
  const int64_t parts = std::max<int64_t>(1, std::min(need, ny * nx / kGatherPartTiles));
  g.zy = (int)std::min(parts, ny);
  g.zx = (int)std::min((parts + g.zy - 1) / g.zy, nx);
  return g;
}

}  // namespace fastvr
