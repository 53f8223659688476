// How many tiles a (expert, row pass) of grouped_flow.hpp is cut into, and what that costs: shared by the kernel and by the
// host code that decides where it runs.
#pragma once
#include <hip/hip_runtime.h>

#include "unit_list.hpp"

namespace moe {
namespace gf {

// Workgroups of a launch, one per compute unit, or 16 units left free for another stream
__host__ __device__ constexpr int workgroups(bool leave_room) { return leave_room ? 240 : 256; }

// Workgroup b runs on XCD b % 8.  The list place of the tile that the id-th take stands for, -1 behind the end.  Each XCD takes a contiguous share of the
// list, the first total % 8 of them one tile more, so that an id has a tile exactly where it is below `total`: a workgroup
// ends at its first take without one, and every later take of anybody has none either.
__host__ __device__ inline int tile_place(int id, int total) {
  if (id >= total) return -1;
  const int xcd = id % gg::kNumXcd, more = total % gg::kNumXcd;
  return xcd * (total / gg::kNumXcd) + (xcd < more ? xcd : more) + id / gg::kNumXcd;
}
// A look-up waits twice for memory (counter, source rows), `pace` k-tiles each: three under load (3 us).  Tiles are looked
// up look_ahead() tiles ahead of time, so that a loader nsb - 1 k-tiles in front finds its tile.
__host__ __device__ constexpr int look_pace(int nk) { return nk >= 16 ? 3 : 1; }
__host__ __device__ constexpr int look_ahead(int nk, int nsb) { return (nsb + 2 * look_pace(nk) + 1 + nk - 1) / nk; }

// Cost of `units` (expert, row pass) pairs of `strips` 16-column output strips in n tiles each: rounds of `wgs` workgroups times
// width, and a quarter of a strip for each tile.  A k-tile has a shortest time (barrier, operand reads, MFMAs of the whole tile shape),
// that of a share of the full width at the HBM rate.
__host__ __device__ inline float tile_cost_of(int units, int wgs, int strips, int n, int bm, int bn, bool gateup) {
  const float full = (float)(bn / (gateup ? 32 : 16));
  const float least = full * (bm >= 160 ? 0.8f : (bm >= 128 ? 0.55f : (bn >= 256 ? 0.35f : 0.5f)));
  const float width = (float)strips / (float)n;
  return (float)((units * n + wgs - 1) / wgs) * ((width > least ? width : least) + 0.25f);
}
// Where a tile's walk over K begins: the matrices of all local experts, one after the other, are cut into regions of
// output columns, and a region's walk begins at its own share of K.  A few large experts have several regions each, and
// then a multiple of as many tiles, so that no tile lies across two.  A function of the expert and the output column
// alone: a row's sums are added in the same order whatever the other rows are and whoever computes them.
__host__ __device__ constexpr int k_regions(int n_local, int bm) { return ((bm >= 128 ? 8 : 16) + n_local - 1) / n_local; }
// (a region's share of K in k-tiles and 1/65536 of one; K <= 2^21, so that K / 64 << 16 fits)
__host__ __device__ inline uint32_t k_step(int n_local, int regions, int nk) {
  return ((uint32_t)nk << 16) / (uint32_t)(n_local * regions);
}
__host__ __device__ inline int k_first(int expert, int nb, int ncb, int regions, uint32_t step) {
  const int region = regions == 1 ? 0 : nb / (ncb / regions);
  return (int)((uint32_t)(expert * regions + region) * step >> 16);
}
// The fewest tiles per unit, and the cheapest number among 64 steps from there on (host code; the kernel prices one per lane).
__host__ __device__ inline int fewest_tiles(int strips, int bn, bool gateup, int regions) {
  const int full = bn / (gateup ? 32 : 16) * regions;
  return (strips + full - 1) / full * regions;
}
inline double tile_cost(int units, int wgs, int n_local, int strips, int bm, int bn, bool gateup, int* tiles) {
  float best = 3e38f;
  const int regions = k_regions(n_local, bm), fewest = fewest_tiles(strips, bn, gateup, regions);
  for (int n = fewest; n < fewest + 64 * regions && n <= strips; n += regions) {
    const float c = tile_cost_of(units, wgs, strips, n, bm, bn, gateup);
    if (c < best) {
      best = c;
      if (tiles != nullptr) *tiles = n;
    }
  }
  return best;
}

}  // namespace gf
}  // namespace moe
