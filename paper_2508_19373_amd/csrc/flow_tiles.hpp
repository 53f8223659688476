// How many tiles a (expert, row pass) of grouped_flow.hpp is cut into, and what that costs: shared by the kernel and by the
// host code that decides where it runs.
#pragma once
#include <hip/hip_runtime.h>

namespace moe {
namespace gf {

constexpr int kRound = 256;  // workgroups of a full launch

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
