// How many tiles a (expert, row pass) of grouped_flow.hpp is cut into, and what that costs: shared by the kernel and by the
// host code that decides where it runs.
#pragma once
#include <hip/hip_runtime.h>

#include "unit_list.hpp"

namespace moe {
namespace gf {

constexpr int kRound = 256;  // workgroups of a full launch

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

// Cost of `units` (expert, row pass) pairs of `strips` 16-column output strips in n tiles each: rounds times width, and a
// quarter of a strip for each tile.  A k-tile has a shortest time (barrier, operand reads, MFMAs of the whole tile shape),
// that of a share of the full width at the HBM rate.
__host__ __device__ inline float tile_cost_of(int units, int strips, int n, int bm, int bn, bool gateup) {
  const float full = (float)(bn / (gateup ? 32 : 16));
  const float least = full * (bm >= 160 ? 0.8f : (bm >= 128 ? 0.55f : (bn >= 256 ? 0.35f : 0.5f)));
  const float width = (float)strips / (float)n;
  return (float)((units * n + kRound - 1) / kRound) * ((width > least ? width : least) + 0.25f);
}
// The fewest tiles per unit, and the cheapest number among 64 from there on (host code; the kernel prices one per lane).
__host__ __device__ inline int fewest_tiles(int strips, int bn, bool gateup) {
  const int full = bn / (gateup ? 32 : 16);
  return (strips + full - 1) / full;
}
inline double tile_cost(int units, int strips, int bm, int bn, bool gateup, int* tiles) {
  float best = 3e38f;
  const int fewest = fewest_tiles(strips, bn, gateup);
  for (int n = fewest; n < fewest + 64 && n <= strips; ++n) {
    const float c = tile_cost_of(units, strips, n, bm, bn, gateup);
    if (c < best) {
      best = c;
      if (tiles != nullptr) *tiles = n;
    }
  }
  return best;
}

}  // namespace gf
}  // namespace moe
