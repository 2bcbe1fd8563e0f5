// Spatial tiling of the latent for tiled inference (FastVR, Sec. 3 overview and
// Sec. 4.1: the DiT runs once per temporal chunk and overlapping 64 x 64 latent
// tile).  Fields are channels-last, x[b, t, y, x, c]; tiles span every frame and
// cut the two spatial axes identically:
//  * placement along an axis of `size`: tile length L = min(tile, size),
//    n = 1 if size <= tile else ceil((size - overlap) / (tile - overlap)) tiles
//    at evenly spaced origins a_k = (k (size - L) + (n - 1) / 2) / (n - 1)
//    (integer division), so a_0 = 0, a_{n-1} = size - L and neighbours overlap
//    by at least `overlap`;
//  * gather: tiles[b, ty * nx + tx, t, iy, ix, c] = x[b, t, a_ty + iy, a_tx + ix, c];
//  * blend: axis weight of tile position i is min(i + 1, L - i, R), R =
//    max(overlap, 1); a tile's weight at a position is the product of its two
//    axis weights, and the field is the weight-normalised sum over the tiles
//    covering the position.  Optionally fused with the one-step update of
//    Eq. 9: z_hat = z_LQ - sigma * blend(v tiles).
// Both kernels are bound by HBM bandwidth.  The gather reads each 16-byte unit of
// the field once and writes it to the tiles that hold it; the blend
// gathers, for each output element, the few tiles covering it (no atomics), with
// the covering tiles of a run of positions found in closed form.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gfx950_ops.h"
#include "launch.h"
#include "tile_plan.h"

namespace fastvr {
namespace {

using namespace dev;

constexpr int kThreads = kTileThreads;

__device__ __forceinline__ int axis_weight(int i, int L, int R) {
  const int m = (i + 1 < L - i) ? i + 1 : L - i;
  return m < R ? m : R;
}

// Gather.  Work item = (field row r = (b * T + t) * Hg + y, segment of seg <= W * U
// consecutive 16-byte units of it, part of its tiles), run by W threads: a wave or
// the workgroup (tile_plan.h).  A thread reads its U units (W apart) once and
// writes them to every tile of its part that holds them; the tiles covering
// the row (along y) and the segment's positions (along x) are two index ranges
// found in closed form, of which part z of zy * zx takes every zy-th and zx-th.
// A tile row is a contiguous run of the field row, so unit u of the field row is
// unit u - ox * C16 of the tile row at origin ox.
// Bound by the HBM writes: each field unit is read once from memory, where one
// workgroup per tile row read every tile's share of it again.  6 tiles of 8 x 64 x
// 64 x 1536 (604 MB written, 200 MB read) 175.6 -> 115.4 us, 7.0 TB/s; 2 x 12
// tiles of 32 x 32 rows, 768 channels 82.8 -> 63.1 us; a single tile (a plain
// copy) 18.5 -> 17.8 us.  Three units a thread: two were 5% slower on the single
// tile, four 1 to 2% on many small tiles; field loads past the caches cost 20%.
// STREAM: stores past the caches.  Not when the tiles of a place are shared among
// workgroups: tile rows then start at any 16 bytes of a line, and the caches
// put the lines together (100 x 100, 48 channels, tiles of 64 one position apart 132
// -> 115 us; 304 x 75, 88 channels, tiles of 11 two apart 65 -> 39 us).
template <typename I, int W, bool STREAM>
__global__ __launch_bounds__(kThreads) void tile_gather_kernel(const u32x4* __restrict__ x, u32x4* __restrict__ tiles,
                                                               int T, int Hg, int Wg, int C16, Axis ay, Axis ax,
                                                               int64_t n_rows, int seg, int zy, int zx) {
  constexpr int U = kGatherUnits, kRows = kThreads / W;
  const int row_units = Wg * C16;
  const int tile_units = ax.L * C16;  // of one tile row
  const int nt = ay.n * ax.n;
  const int64_t tile_rows = (int64_t)T * ay.L;
  const int u_begin = blockIdx.x * seg;
  const int u_end = min(u_begin + seg, row_units);
  const int tx_hi = last_start_le<I>(ax, (u_end - 1) / C16);
  const int ty_part = (int)blockIdx.z % zy, tx_lo = first_end_gt<I>(ax, u_begin / C16) + (int)blockIdx.z / zy;
  // W >= 64: one row per wave
  const int sub = W == kThreads ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.y);
  for (int64_t r = (int64_t)blockIdx.y * kRows + sub; r < n_rows; r += (int64_t)gridDim.y * kRows) {
    u32x4 val[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int u = u_begin + k * W + (int)threadIdx.x;
      if (u < u_end) val[k] = x[r * row_units + u];
    }
    const I rr = (I)r;
    const int y = (int)(rr % (I)Hg);
    const I bt = rr / (I)Hg;
    const int t = (int)(bt % (I)T);
    const int64_t b = (int64_t)(bt / (I)T);
    const int ty_hi = last_start_le<I>(ay, y);
    for (int ty = first_end_gt<I>(ay, y) + ty_part; ty <= ty_hi; ty += zy) {
      const int64_t row0 = ((b * nt + ty * ax.n) * T + t) * ay.L + (y - origin_t<I>(ay, ty));  // tile row for tx = 0
      for (int tx = tx_lo; tx <= tx_hi; tx += zx) {
        const int u0 = origin_t<I>(ax, tx) * C16;
        u32x4* dst = tiles + (row0 + (int64_t)tx * tile_rows) * tile_units;
#pragma unroll
        for (int k = 0; k < U; ++k) {
          const int u = u_begin + k * W + (int)threadIdx.x, v = u - u0;
          if (u < u_end && v >= 0 && v < tile_units) {
            if (STREAM)
              __builtin_nontemporal_store(val[k], dst + v);
            else
              dst[v] = val[k];
          }
        }
      }
    }
  }
}

// Work item = (output row r = (b * T + t) * Hg + y, segment of kThreads * U
// consecutive units of that row); a unit is 4 channels of one position (16 bytes
// of fp32).  The tiles covering the row (along y) and the segment's positions
// (along x) are two index ranges found in closed form once per item; a thread
// then forms its U units (kThreads apart), issuing the loads of all U units
// from one tile before using any.  With Z (fused Eq. 9) the output is
// z - sigma * blend, z bf16.
template <bool Z, typename I, int U, bool STREAM>
__global__ __launch_bounds__(kThreads) void tile_blend_kernel(const float* __restrict__ tiles,
                                                              const uint16_t* __restrict__ z, float* __restrict__ out,
                                                              float neg_sigma, int T, int Hg, int Wg, int C, Axis ay,
                                                              Axis ax, int R, int64_t n_rows) {
  const int C4 = C / 4;
  const int row_units = Wg * C4;
  const int nt = ay.n * ax.n;
  const int64_t tile_rows = (int64_t)T * ay.L;  // rows of one tile
  const int u_begin = blockIdx.x * (kThreads * U);
  const int u_end = min(u_begin + kThreads * U, row_units);
  int xg[U], c4[U];
  bool ok[U];
#pragma unroll
  for (int k = 0; k < U; ++k) {
    const int u = u_begin + k * kThreads + (int)threadIdx.x;
    ok[k] = u < u_end;
    xg[k] = ok[k] ? u / C4 : 0;
    c4[k] = u - xg[k] * C4;
  }
  const int tx_lo = first_end_gt<I>(ax, u_begin / C4), tx_hi = last_start_le<I>(ax, (u_end - 1) / C4);
  for (int64_t r = blockIdx.y; r < n_rows; r += gridDim.y) {
    const I rr = (I)r;
    const int y = (int)(rr % (I)Hg);
    const I bt = rr / (I)Hg;
    const int t = (int)(bt % (I)T);
    const int64_t b = (int64_t)(bt / (I)T);
    f32x4 acc[U];
    float wsum[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
      acc[k] = f32x4{0.f, 0.f, 0.f, 0.f};
      wsum[k] = 0.f;
    }
    const int ty_hi = last_start_le<I>(ay, y);
    for (int ty = first_end_gt<I>(ay, y); ty <= ty_hi; ++ty) {
      const int iy = y - origin_t<I>(ay, ty);
      const int wy = axis_weight(iy, ay.L, R);
      const int64_t row0 = ((b * nt + ty * ax.n) * T + t) * ay.L + iy;  // tile row for tx = 0
      for (int tx = tx_lo; tx <= tx_hi; ++tx) {
        const int ox = origin_t<I>(ax, tx);
        const float* trow = tiles + (row0 + (int64_t)tx * tile_rows) * ax.L * C;
        f32x4 val[U];
        float w[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
          const int ix = xg[k] - ox;
          val[k] = f32x4{0.f, 0.f, 0.f, 0.f};
          w[k] = 0.f;
          if (ok[k] && ix >= 0 && ix < ax.L) {
            w[k] = (float)(wy * axis_weight(ix, ax.L, R));
            const f32x4* src = reinterpret_cast<const f32x4*>(trow + (int64_t)ix * C + 4 * c4[k]);
            val[k] = STREAM ? __builtin_nontemporal_load(src) : *src;
          }
        }
#pragma unroll
        for (int k = 0; k < U; ++k) {
          acc[k].x = __builtin_fmaf(w[k], val[k].x, acc[k].x);
          acc[k].y = __builtin_fmaf(w[k], val[k].y, acc[k].y);
          acc[k].z = __builtin_fmaf(w[k], val[k].z, acc[k].z);
          acc[k].w = __builtin_fmaf(w[k], val[k].w, acc[k].w);
          wsum[k] += w[k];
        }
      }
    }
#pragma unroll
    for (int k = 0; k < U; ++k) {
      if (!ok[k]) continue;
      f32x4 res = {acc[k].x / wsum[k], acc[k].y / wsum[k], acc[k].z / wsum[k], acc[k].w / wsum[k]};
      const int64_t o = (r * Wg + xg[k]) * C + 4 * c4[k];
      if (Z) {
        const uint64_t zz = *reinterpret_cast<const uint64_t*>(z + o);
        const __bf16* zb = reinterpret_cast<const __bf16*>(&zz);
        res.x = __builtin_fmaf(neg_sigma, res.x, (float)zb[0]);
        res.y = __builtin_fmaf(neg_sigma, res.y, (float)zb[1]);
        res.z = __builtin_fmaf(neg_sigma, res.z, (float)zb[2]);
        res.w = __builtin_fmaf(neg_sigma, res.w, (float)zb[3]);
      }
      __builtin_nontemporal_store(res, reinterpret_cast<f32x4*>(out + o));
    }
  }
}

Axis make_axis(int64_t size, int64_t tile, int64_t overlap) {
  const TileAxis t = tile_axis(size, tile, overlap);
  return Axis{(int)t.n, (int)t.len, (int)(size - t.len)};
}

// 32-bit index arithmetic when the row index and every origin numerator (below
// n * size along each axis) stay below 2^32.
bool narrow_index(int64_t rows, const Axis& ay, const Axis& ax, int64_t Hg, int64_t Wg) {
  const int64_t lim = int64_t(1) << 32;
  return rows < lim && (int64_t)ay.n * Hg < lim && (int64_t)ax.n * Wg < lim;
}

dim3 row_grid(int64_t row_units, int64_t rows, int units) {
  return dim3((unsigned)((row_units + kThreads * units - 1) / (kThreads * units)),
              (unsigned)(rows < 65535 ? rows : 65535));
}

}  // namespace

hipError_t launch_tile_gather(const void* x, void* tiles, int64_t B, int64_t T, int64_t Hg, int64_t Wg, int64_t C,
                              int64_t tile, int64_t overlap, hipStream_t stream) {
  const Axis ay = make_axis(Hg, tile, overlap), ax = make_axis(Wg, tile, overlap);
  const int64_t rows = B * T * Hg;
  const GatherGrid g = gather_grid(rows, Wg, C / 8, ay, ax);
  const dim3 grid((unsigned)g.segments, (unsigned)g.row_groups, (unsigned)(g.zy * g.zx));
  const dim3 block(g.width, kThreads / g.width);
  const u32x4* xp = static_cast<const u32x4*>(x);
  u32x4* tp = static_cast<u32x4*>(tiles);
#define FASTVR_GATHER_LAUNCH(IT, WV, SV)                                                                             \
  hipLaunchKernelGGL((tile_gather_kernel<IT, WV, SV>), grid, block, 0, stream, xp, tp, (int)T, (int)Hg, (int)Wg, \
                     (int)(C / 8), ay, ax, rows, g.seg, g.zy, g.zx)
#define FASTVR_GATHER_INDEX(WV, SV)                        \
  do {                                                     \
    if (narrow) FASTVR_GATHER_LAUNCH(uint32_t, WV, SV);    \
    else FASTVR_GATHER_LAUNCH(uint64_t, WV, SV);           \
  } while (0)
  const bool narrow = narrow_index(rows, ay, ax, Hg, Wg), shared = g.zy * g.zx > 1;
  if (g.width == 64) {
    if (shared) FASTVR_GATHER_INDEX(64, false);
    else FASTVR_GATHER_INDEX(64, true);
  } else {
    if (shared) FASTVR_GATHER_INDEX(kThreads, false);
    else FASTVR_GATHER_INDEX(kThreads, true);
  }
#undef FASTVR_GATHER_INDEX
#undef FASTVR_GATHER_LAUNCH
  return hipGetLastError();
}

hipError_t launch_tile_blend(const float* tiles, const void* z_lq, float* out, float sigma, int64_t B, int64_t T,
                             int64_t Hg, int64_t Wg, int64_t C, int64_t tile, int64_t overlap, hipStream_t stream) {
  const Axis ay = make_axis(Hg, tile, overlap), ax = make_axis(Wg, tile, overlap);
  const int64_t rows = B * T * Hg;
  const int R = overlap > 1 ? (int)overlap : 1;
  const int64_t row_units = Wg * (C / 4);
  const bool narrow = narrow_index(rows, ay, ax, Hg, Wg);
  // Up to 64 MB of tiles are mostly still in the 256 MB Infinity Cache when the call
  // follows the one that produced them, and are read through the caches; larger
  // ones, each read exactly once, past them.  Two units a thread (more waves), four
  // beyond 320 MB.  Measured with four inputs in turn, against non-temporal loads
  // of four units for all sizes: 47 MB of tiles 15.8 -> 11.8 us (14.7 past the
  // caches); 201 MB 62.4 -> 47.7 us (51.4 through them); 277 MB 74.0 -> 69.7 us; at
  // 390 MB two and four units are equal, at 1.2 GB four take 257 and two 266 us.
  const int64_t tile_bytes = B * ay.n * ax.n * T * ay.L * ax.L * C * 4;
  const bool cached = tile_bytes <= ((int64_t)64 << 20), four = tile_bytes > ((int64_t)320 << 20);
  const dim3 grid = row_grid(row_units, rows, four ? 4 : 2);
  const uint16_t* zp = static_cast<const uint16_t*>(z_lq);
  const float ns = z_lq != nullptr ? -sigma : 0.f;
#define FASTVR_BLEND_LAUNCH(ZV, IT, UV, SV)                                                                             \
  hipLaunchKernelGGL((tile_blend_kernel<ZV, IT, UV, SV>), grid, dim3(kThreads), 0, stream, tiles, zp, out, ns, (int)T, \
                     (int)Hg, (int)Wg, (int)C, ay, ax, R, rows)
#define FASTVR_BLEND_INDEX(ZV, UV, SV)                      \
  do {                                                      \
    if (narrow) FASTVR_BLEND_LAUNCH(ZV, uint32_t, UV, SV);  \
    else FASTVR_BLEND_LAUNCH(ZV, uint64_t, UV, SV);         \
  } while (0)
  if (z_lq != nullptr) {
    if (four) FASTVR_BLEND_INDEX(true, 4, true);
    else if (cached) FASTVR_BLEND_INDEX(true, 2, false);
    else FASTVR_BLEND_INDEX(true, 2, true);
  } else {
    if (four) FASTVR_BLEND_INDEX(false, 4, true);
    else if (cached) FASTVR_BLEND_INDEX(false, 2, false);
    else FASTVR_BLEND_INDEX(false, 2, true);
  }
#undef FASTVR_BLEND_INDEX
#undef FASTVR_BLEND_LAUNCH
  return hipGetLastError();
}

}  // namespace fastvr
