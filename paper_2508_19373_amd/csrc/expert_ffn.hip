// Expert networks on the permuted rows (paper, "MoE Model Architectures": the Expert module's
// parallel expert networks, evaluated only for the tokens the gating network sent to them;
// "Tensor Parallelism": a shard may hold only a slice of the intermediate dimension, in which
// case the result is the unreduced partial sum).
//
// Two grouped GEMMs, both "NT" (activations and weights are K-contiguous):
//   GEMM1  h[r, i]  = silu(x_r . Wg_e[i,:]) * (x_r . Wu_e[i,:])      K = H,   N = I_s (gate+up fused)
//   GEMM2  y[r, n]  = h_r . Wd_e[n,:]                                K = I_s, N = H
// bf16 operands, fp32 accumulators.  Three kernel families cover the two regimes the paper
// distinguishes ("Generative Inference"): grouped_gemm.hpp (tiled, LDS-DMA, MFMA-bound) for
// prefill-sized groups; for decode-sized groups grouped_flow.hpp (tiles whose weight stream never stops, HBM-bound; flow_plan
// below says where) and grouped_walk.hpp (weight streaming in passes of 16 or 32 rows; grouped_stream.hpp for the K extents it
// is not instantiated for).  Each of the two GEMMs picks its family on its own (flow_plan, then the estimate of prefer_walk).  In both, the work list is derived on the
// device from expert_offsets without a host round trip.
#include "flow_tiles.hpp"
#include "grouped_gemm.hpp"
#include "grouped_stream.hpp"
#include "grouped_walk.hpp"
#include "moe_internal.hpp"

#include <cmath>

namespace moe {
namespace {

// Rows the fullest local expert is planned for.  A shard that holds every expert gets exactly the
// capacity, and only its spread over the experts is open: the average plus two sigma.  An
// expert-parallel shard's share of the batch follows the routing ("Expert Parallelism": load
// imbalance), and the shard that sets the latency of the step is the one that got more than its
// share, so it is planned for twice the balanced share (under Zipf(1.2) popularity the first of four
// shards receives 55 % of the rows, 2.2 times a quarter), never more than the whole capacity.
inline double planned_rows_hi(int cap_rows, int est_rows, int n_local) {
  double avg = (double)est_rows / n_local;
  if (n_local == 1 && est_rows == cap_rows) return avg;  // one expert that takes every row
  if (est_rows < cap_rows) avg = fmin(2.0 * avg, (double)cap_rows / n_local);
  return avg + 2.0 * sqrt(avg);
}

// Row-block height of the tiled kernels for a call without tall row blocks (tall_blocks_allowed comes first: it takes
// the band around 273 rows up to 305, given K extents of 1024): 160 (the one-height list) or 256.
// The 160-row tiling pays where it saves the second stream of an expert's weights (or a padded
// 256-row tile) without adding a block: with the rows per expert just below a multiple of 160.
// Measured, gate/up + down projection in us, 256-row tiling against 160-row tiling, by average rows
// per expert: Qwen1.5-MoE (60 experts) 102: 243 / 243; 136: 275 / 254; 170: 296 / 359; 204: 301 / 392;
// 238: 323 / 397; 273: 441 / 402; 307: 488 / 435; 341: 497 / 522; 409: 512 / 534; Qwen2-57B (64
// experts) 128: 830 / 753; 192: 895 / 1141; 256: 1206 / 1172; 320: 1593 / 1408; 384: 1518 / 1645.
// With 30 local experts (273 rows each) the two are equal, with 8 large experts the 160-row tiling
// loses a fifth, hence the expert count in the rule.
#ifndef MOE_EVEN_MODE
#define MOE_EVEN_MODE 0  // 1: always 160, 2: never (tuning builds)
#endif
inline bool prefer_even(int est_rows, int n_local, int H, int I_s) {
  (void)H;
  (void)I_s;
  if (MOE_EVEN_MODE != 0) return MOE_EVEN_MODE == 1;
  const double avg = (double)est_rows / n_local;
  return n_local >= 32 && ((avg >= 115.0 && avg <= 148.0) || (avg >= 255.0 && avg <= 330.0));
}

// Whether a tiled call's full row blocks may take their expert's remainder (where the list then has tall blocks:
// dealing_pays, expects_tall_blocks).  From 150 rows per expert on: below, hardly an expert has a full block.  Measured, gate/up +
// down projection in us on one box, without / with: Mixtral (8 experts) 1053 rows each 1653 + 833 / 1419 + 722, 1088:
// 1667 + 836 / 1463 + 744, 1152: 1714 + 862 / 1569 + 845; its TP=4 slice 2068: 738 + 430 / 693 + 381; counts as a router
// spreads 4096 tokens 1538 + 780 / 1461 + 735.  No remainders at all, when such launches still ran the kernel with tall
// blocks: 1024 rows 1353 + 675 / 1363 + 675, TP=4 slice 2048 down projection 370 / 383, 2304 gate/up 752 / 760.  Qwen1.5-MoE (60
// experts, the 160-row tiling before) 256: 262 + 144 / 216 + 123, 286: 262 + 150 / 234 + 134, spread about 273: 258 +
// 154 / 223 + 144.  Not in the 160-row tiling's band above 305 rows per expert: from there on most experts have more than
// the 304 rows of one tall block, so the remainder tiles are back.  160-row / tall: Qwen1.5-MoE 300 255 + 151 / 252 + 154,
// 320 285 + 169 / 295 + 173, 330 298 + 169 / 311 + 193; Qwen2-57B 300 794 + 467 / 790 + 461, 310 840 + 505 / 874 + 516, 320
// 899 + 510 / 943 + 564, 340 (256-row before) 1015 + 617 / 1000 + 595; its EP=2 shard 310 423 + 249 / 456 + 263.  Both K extents
// from 1024 on: on a shorter walk the larger kernel costs more than it saves.  H = I_s = 768: 8 experts of 1040 rows 29.5 +
// 29.2 / 31.2 + 30.6, 16 of 1050 54.1 + 30.3 / 55.4 + 31.5, 64 of 280 68.8 + 41.0 / 63.8 + 38.4 (76.0 + 41.9 in blocks of 160); 1024: 16 of 1050
// 78.8 + 53.6 / 71.7 + 44.1, 64 of 280 116 + 65 / 106 + 59 (122 + 72).  A tall block addresses its operands with
// 32-bit byte offsets from its first row, so 304 rows of either K extent have to fit.
bool tall_blocks_allowed(int est_rows, int n_local, int H, int I_s) {
  constexpr uint64_t kMaxK = gg::kBufBytes / (2 * (256 + 16 * gg::kMaxExtra));
  if ((uint64_t)H > kMaxK || (uint64_t)I_s > kMaxK) return false;
  const double avg = (double)est_rows / n_local;
  if (avg > 305.0 && prefer_even(est_rows, n_local, H, I_s)) return false;
  return avg >= 150.0 && H >= 1024 && I_s >= 1024;
}

// Whether a GEMM's list is expected to have tall blocks: the list itself, for a routing that spreads as a balanced router does
// (the experts at the quantiles of a normal distribution) or, on an expert-parallel shard, for one that got what it is
// planned for.
// A launch without any takes the plain kernel: the one with tall blocks costs it a few per cent (shared expert of 333
// rows, 88 tiles: gate/up 53.1 -> 56.6 us; 8 experts of 160 rows, down projection 228 -> 233; 4 of 600 rows 317 -> 328).
bool expects_tall_blocks(int cap_rows, int est_rows, int n_local, int ncb, int nk, bool sliced) {
  const bool exact = n_local == 1 && est_rows == cap_rows;  // one expert that takes every row
  const double avg = (double)est_rows / n_local;
  int32_t offsets[MOE_MAX_EXPERTS + 1];
  auto tall = [&](double rows, bool cut) {
    double at = 0.0;
    offsets[0] = 0;
    for (int e = 0; e < n_local; ++e) {
      const double u = (2 * e + 1.0) / n_local - 1.0, u2 = u * u, u8 = u2 * u2 * u2 * u2;
      at += rows + sqrt(rows) * u * (1.25 + 0.2 * u2 + 0.95 * u8);  // normal quantile, within 0.2 for up to 64 experts
      offsets[e + 1] = (int32_t)fmin(at + 0.5, 1 << 30);
    }
    return gg::count_tiles(offsets, n_local, ncb, cut ? gg::sliced_pad_from(nk) : gg::kPadLowTiles, true, nk,
                           cut ? gg::max_k_slices(nk * gg::BK) : 0)
        .tall;
  };
  // (not for a finer cut either: the lookup costs it more, shared expert of 4100 rows, down projection 109 us plain, 116)
  if (exact) return !sliced && tall(avg, false);
  // (a shard's planned share not for a finer cut, which hangs on a tile more or less: 4 of 8 experts of 256 rows, 187 us plain, 199)
  return tall(avg, sliced) || (est_rows < cap_rows && tall(fmin(2.0 * avg, (double)cap_rows / n_local), false));
}

// Whether the tiles of a gate/up projection begin their walk over K apart (gemm_tile): where rows are a multiple of 4 KB and
// the weights, not the matrix cores, set the pace.  Measured from one place / spread, us: TP=4 slice of Mixtral, 160 rows
// per expert 119 / 111, 300: 194 / 182; Qwen1.5-MoE 256: 210 / 194, 272: 220 / 206; 64 experts of 280 rows, K = 2048, 257 /
// 242; at the power limit it costs a little (Mixtral 1024 rows 1383 / 1391, 1040: 1432 / 1458), and so does the arithmetic (the
// choice made in the kernel: TP=4 slice 2048 rows 676 -> 692 from one place), hence kernels of their own; on other K nothing
// changes (Qwen2-57B, K = 3584, 553 / 549).  The 160-row tiling gains 1 %, the down projections lose (Mixtral 1024 rows 678 / 689).
inline bool spread_k(int est_rows, int n_local, int K) { return K % 2048 == 0 && est_rows <= 512 * n_local; }

// Prefill-sized groups: LDS-DMA kernel, 256-column tiles of 256 / 128 / 64 rows, or the kernel whose full row blocks may take
// their expert's remainder (tall_gemms).
template <int BN>
hipError_t launch_pair_dlds(const void* x_perm, RowMap rows, const int32_t* expert_offsets, int cap_rows, int est_rows, int n_local, int H,
                            int I_s, const void* w_gate, const void* w_up, const void* w_down, void* h_ws,
                            void* y_perm, void* workspace, uint32_t flags, hipStream_t stream) {
  const bool y_bf16 = (flags & MOE_Y_PERM_BF16) != 0;
  const dim3 block(256);
  static_assert(BN == 256, "tall_gemms counts column blocks of 256 weight rows");
  const uint16_t* xp = static_cast<const uint16_t*>(x_perm);
  uint16_t* hw = static_cast<uint16_t*>(h_ws);
  auto grid_for = [&](int ncb) { return dim3((unsigned)gg::max_grid(cap_rows, n_local, ncb)); };
  if (!(flags & MOE_FFN_SKIP_GATEUP)) {
    const int ncb = (I_s + BN / 2 - 1) / (BN / 2);
    const bool spread = spread_k(est_rows, n_local, H);
    const auto kernel = tall_gemms(cap_rows, est_rows, n_local, H, I_s, kTallGateUp)
                            ? (spread ? gg::grouped_gemm_spread_tall_kernel<BN> : gg::grouped_gemm_tall_kernel<BN, true, uint16_t, false>)
                            : (spread ? gg::grouped_gemm_spread_kernel<BN> : gg::grouped_gemm_dlds_kernel<BN, true, uint16_t, false>);
    hipLaunchKernelGGL(kernel, grid_for(ncb), block, 0, stream, xp,
                       expert_offsets, n_local, cap_rows, static_cast<const uint16_t*>(w_gate),
                       static_cast<const uint16_t*>(w_up), I_s, H, hw, ncb, static_cast<uint16_t*>(nullptr), 0, rows);
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
  }
  if (flags & MOE_FFN_SKIP_DOWN) return hipSuccess;
  const int ncb = (H + BN - 1) / BN;
  const gg::SlicePlan sp =
      y_bf16 || workspace == nullptr ? gg::SlicePlan{1, 0} : gg::slice_plan(cap_rows, ncb, I_s);
  const bool tall =
      tall_gemms(cap_rows, est_rows, n_local, H, I_s, y_bf16 || workspace == nullptr ? kTallDownBf16 : kTallDown) != 0;
  if (y_bf16) {
    const auto kernel = tall ? gg::grouped_gemm_tall_kernel<BN, false, uint16_t, false>
                             : gg::grouped_gemm_dlds_kernel<BN, false, uint16_t, false>;
    hipLaunchKernelGGL(kernel, grid_for(ncb), block, 0, stream, hw,
                       expert_offsets, n_local, cap_rows, static_cast<const uint16_t*>(w_down),
                       static_cast<const uint16_t*>(nullptr), H, I_s, static_cast<uint16_t*>(y_perm), ncb,
                       static_cast<uint16_t*>(nullptr), 0, RowMap{nullptr, 1});
    return hipGetLastError();
  }
  float* yp = static_cast<float*>(y_perm);
  float* ws = static_cast<float*>(workspace);
  const uint16_t* wd = static_cast<const uint16_t*>(w_down);
  if (sp.max_slices == 1) {
    const auto kernel = tall ? gg::grouped_gemm_tall_kernel<BN, false, float, false>
                             : gg::grouped_gemm_dlds_kernel<BN, false, float, false>;
    hipLaunchKernelGGL(kernel, grid_for(ncb), block, 0, stream, hw,
                       expert_offsets, n_local, cap_rows, wd, static_cast<const uint16_t*>(nullptr), H, I_s, yp, ncb,
                       static_cast<float*>(nullptr), 0, RowMap{nullptr, 1});
    return hipGetLastError();
  }
  const auto kernel = tall ? gg::grouped_gemm_tall_kernel<BN, false, float, true>
                           : gg::grouped_gemm_dlds_kernel<BN, false, float, true>;
  hipLaunchKernelGGL(kernel,
                     dim3(gg::sliced_grid(cap_rows, n_local, ncb)), block, 0, stream, hw, expert_offsets, n_local,
                     cap_rows, wd, static_cast<const uint16_t*>(nullptr), H, I_s, ws, ncb, yp, sp.max_slices,
                     RowMap{nullptr, 1});
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  const auto sum = tall ? gg::sum_sliced_kernel<true> : gg::sum_sliced_kernel<false>;
  hipLaunchKernelGGL(sum, dim3(192, (H + 1023) / 1024), dim3(256), 0, stream, ws, expert_offsets, n_local, ncb,
                     I_s / gg::BK, sp.max_slices, H, yp);
  return hipGetLastError();
}

// A few hundred rows per expert: tiles of 160 rows from the one-height work list (unit_list_even.hpp).
hipError_t launch_pair_even(const void* x_perm, RowMap rows, const int32_t* expert_offsets, int cap_rows, int n_local,
                            int H, int I_s, const void* w_gate, const void* w_up, const void* w_down, void* h_ws,
                            void* y_perm, uint32_t flags, hipStream_t stream) {
  const dim3 block(256);
  uint16_t* hw = static_cast<uint16_t*>(h_ws);
  if (!(flags & MOE_FFN_SKIP_GATEUP)) {
    const int ncb = (I_s + 127) / 128;
    hipLaunchKernelGGL((gg::grouped_gemm_even_kernel<256, true, uint16_t>),
                       dim3((unsigned)gg::even_max_ids(cap_rows, n_local, ncb)), block, 0, stream,
                       static_cast<const uint16_t*>(x_perm), expert_offsets, n_local, cap_rows,
                       static_cast<const uint16_t*>(w_gate), static_cast<const uint16_t*>(w_up), I_s, H, hw, ncb, rows);
    const hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
  }
  if (flags & MOE_FFN_SKIP_DOWN) return hipSuccess;
  const int ncb = (H + 255) / 256;
  const dim3 grid((unsigned)gg::even_max_ids(cap_rows, n_local, ncb));
  if (flags & MOE_Y_PERM_BF16)
    hipLaunchKernelGGL((gg::grouped_gemm_even_kernel<256, false, uint16_t>), grid, block, 0, stream, hw, expert_offsets,
                       n_local, cap_rows, static_cast<const uint16_t*>(w_down), static_cast<const uint16_t*>(nullptr), H,
                       I_s, static_cast<uint16_t*>(y_perm), ncb, RowMap{nullptr, 1});
  else
    hipLaunchKernelGGL((gg::grouped_gemm_even_kernel<256, false, float>), grid, block, 0, stream, hw, expert_offsets,
                       n_local, cap_rows, static_cast<const uint16_t*>(w_down), static_cast<const uint16_t*>(nullptr), H,
                       I_s, static_cast<float*>(y_perm), ncb, RowMap{nullptr, 1});
  return hipGetLastError();
}

// Decode-sized groups, register-resident activations (grouped_walk.hpp).  Returns false when the
// K extent is not one of the instantiated (wavefronts x steps) splits.
constexpr int kWalkSlots = 512;  // 8-wavefront workgroups resident at once with MT = 1 (2 per CU); half of it
                                  // with MT = 2 or 16 wavefronts (1 per CU)

template <int MT, bool GATEUP>
bool launch_walk(const gw::WalkPlan& plan, const uint16_t* A, const int32_t* expert_offsets, int n_local,
                 const uint16_t* Wa, const uint16_t* Wb, int n_out, int K, void* C, int cap_rows, RowMap rows,
                 bool leave_room, hipStream_t stream) {
  // as many workgroups as are resident at once; the kernel cuts its work list into that many ranges
  int n_wg = (MT == 1 && plan.nw < 16 ? kWalkSlots : kWalkSlots / 2) / plan.slices;
  if (leave_room) n_wg = n_wg * 15 / 16;  // 16 compute units stay free for a tiled call on another stream
  n_wg = n_wg < 1 ? 1 : n_wg;
  const dim3 grid(n_wg, 1, plan.slices);
#define MOE_WALK(NW, ST)                                                                                        \
  if (plan.nw == NW && plan.steps == ST) {                                                                      \
    hipLaunchKernelGGL((gw::grouped_walk_kernel<NW, ST, MT, GATEUP>), grid, dim3(NW * 64), 0, stream, A,        \
                       expert_offsets, Wa, Wb, n_out, K, C, n_local, cap_rows, rows);                               \
    return true;                                                                                                \
  }
  if constexpr (MT == 1) {
    MOE_WALK(16, 14)
    MOE_WALK(16, 11)
  }
  if constexpr (MT == 1 || !GATEUP) {  // with 32 rows per pass only the down projection fits sixteen wavefronts
    MOE_WALK(16, 8)
    MOE_WALK(16, 7)
    MOE_WALK(16, 5)
    MOE_WALK(16, 4)
  }
  MOE_WALK(8, 16)
  MOE_WALK(8, 14)
  MOE_WALK(8, 11)
  MOE_WALK(8, 10)
  MOE_WALK(8, 8)
  MOE_WALK(8, 7)
  MOE_WALK(8, 5)
  if constexpr (MT == 2) MOE_WALK(8, 2)
  MOE_WALK(4, 11)
  MOE_WALK(4, 10)
  MOE_WALK(4, 8)
  MOE_WALK(4, 5)
#undef MOE_WALK
  return false;
}

template <int MT>
hipError_t launch_pair_decode(const void* x_perm, RowMap rows, const int32_t* expert_offsets, int cap_rows, int n_local, int H,
                              int I_s, const void* w_gate, const void* w_up, const void* w_down, void* h_ws,
                              void* y_perm, void* workspace, uint32_t flags, hipStream_t stream) {
  const bool y_bf16 = (flags & MOE_Y_PERM_BF16) != 0;
  const uint16_t* xp = static_cast<const uint16_t*>(x_perm);
  uint16_t* hw = static_cast<uint16_t*>(h_ws);
  if (n_local > 65535) return hipErrorInvalidValue;
  if (!(flags & MOE_FFN_SKIP_GATEUP)) {
    const gw::WalkPlan p1 = gw::plan_for(H, MT);
    bool done = false;
    if (p1.nw != 0 && p1.slices == 1 && I_s % 16 == 0)
      done = launch_walk<MT, true>(p1, xp, expert_offsets, n_local, static_cast<const uint16_t*>(w_gate),
                                   static_cast<const uint16_t*>(w_up), I_s, H, hw, cap_rows, rows,
                                   (flags & MOE_FFN_LEAVE_ROOM) != 0, stream);
    if (!done) {
      const dim3 grid((I_s + gs::kStripN - 1) / gs::kStripN, n_local);
      hipLaunchKernelGGL((gs::grouped_stream_kernel<MT, true, uint16_t>), grid, dim3(gs::kWaves * 64), 0, stream, xp,
                         expert_offsets, static_cast<const uint16_t*>(w_gate), static_cast<const uint16_t*>(w_up),
                         I_s, H, hw, rows);
    }
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
  }
  if (flags & MOE_FFN_SKIP_DOWN) return hipSuccess;
  const gw::WalkPlan p2 = gw::plan_for(I_s, MT, true);
  if (!y_bf16 && p2.nw != 0 && H % 16 == 0 && (p2.slices == 1 || workspace != nullptr)) {
    void* out = p2.slices == 1 ? y_perm : workspace;
    if (launch_walk<MT, false>(p2, hw, expert_offsets, n_local, static_cast<const uint16_t*>(w_down),
                               static_cast<const uint16_t*>(nullptr), H, I_s, out, cap_rows, RowMap{nullptr, 1},
                               (flags & MOE_FFN_LEAVE_ROOM) != 0, stream)) {
      hipError_t err = hipGetLastError();
      if (err != hipSuccess || p2.slices == 1) return err;
      hipLaunchKernelGGL(gw::sum_slices_kernel, dim3(64), dim3(256), 0, stream, static_cast<const float*>(workspace),
                         expert_offsets, n_local, cap_rows, H, p2.slices, static_cast<float*>(y_perm));
      return hipGetLastError();
    }
  }
  const dim3 grid((H + gs::kStripN - 1) / gs::kStripN, n_local);
  if (y_bf16)
    hipLaunchKernelGGL((gs::grouped_stream_kernel<MT, false, uint16_t>), grid, dim3(gs::kWaves * 64), 0, stream, hw,
                       expert_offsets, static_cast<const uint16_t*>(w_down), static_cast<const uint16_t*>(nullptr),
                       H, I_s, static_cast<uint16_t*>(y_perm), RowMap{nullptr, 1});
  else
    hipLaunchKernelGGL((gs::grouped_stream_kernel<MT, false, float>), grid, dim3(gs::kWaves * 64), 0, stream, hw,
                       expert_offsets, static_cast<const uint16_t*>(w_down), static_cast<const uint16_t*>(nullptr),
                       H, I_s, static_cast<float*>(y_perm), RowMap{nullptr, 1});
  return hipGetLastError();
}

// MT = 1 (16 activation rows per pass) when the fullest expert is expected to stay within 16 rows
// (certain when the whole capacity is 16 rows): it keeps twice the bytes in flight, and an expert
// with more rows only pays another pass over its own weights.
inline int decode_mt(int cap_rows, int est_rows, int n_local) {
  return (cap_rows <= 16 || planned_rows_hi(cap_rows, est_rows, n_local) <= 16.0) ? 1 : 2;
}

// Which kernel family runs one of the two GEMMs: the weight-streaming walk (decode regime) or the
// tiled LDS-DMA kernel (prefill regime).  A few rows per expert are bound by streaming the
// weights once, many rows by the matrix cores; in between, what decides is how often the walk has
// to re-stream an expert (one pass per 16 or 32 rows) against how many tiles the tiled kernel can
// spread over the compute units (the down projection of a single shared expert has H / 256 = 14
// column blocks per row block: 14 CUs, which is why such a launch is also cut along K).
// Estimates in seconds, from measured rates on MI355X:
//   walk   passes * (bytes / rate + 5 us), rate 6.0 / 5.4 TB/s (GEMM1 / GEMM2) at 16 rows per pass,
//          5.3 / 4.9 TB/s at 32, 3 TB/s for K extents only the generic streaming kernel covers;
//          passes from the rows of the fullest expert (planned_rows_hi);
//   tiled  rounds * (tile time + 8 us), rounds = tiles * slices / 256, at least one; tile time is the
//          larger of streaming the tile's weight panel latency-bound (45 GB/s per compute unit) and
//          its MFMA pace (1.3 us per k-tile of a full 256-row tile); never faster than 1.2 PFLOP/s
//          overall.  What HBM allows when all compute units stream at once: for the gate/up
//          projection all panels together at 5.7 TB/s + 4 us (measured 5.4-5.9 TB/s); for the down
//          projection the per-unit rate is capped at 5.4 TB/s / busy units inside the tile time
//          (its partial sums and their addition ride on the 8 us).
// (Measured, Mixtral TP=4 shard at 48-64 tokens: gate/up streaming with 32 rows per pass 90.5-91.8 us,
// tiled 86.2-86.6; with 16 rows per pass at 16-32 tokens 80.5-81.8 against 85.7.  Qwen1.5 down
// projection at 64-128 tokens: streaming 68.0 / 73.7 us, tiled 61.8 / 66.0.)
inline bool prefer_walk(int cap_rows, int est_rows, int n_local, int n_out, int K, bool gateup) {
  const double mats = gateup ? 2.0 : 1.0;
  const bool exact = n_local == 1 && est_rows == cap_rows;  // one expert that takes every row
  const double rows_hi = planned_rows_hi(cap_rows, est_rows, n_local);
  const int mt = decode_mt(cap_rows, est_rows, n_local);
  const double passes = ceil(rows_hi / (16.0 * mt));
  const double bytes = mats * n_local * (double)n_out * K * 2.0;
  const gw::WalkPlan wp = gw::plan_for(K, mt, !gateup);
  const double rate = wp.nw == 0 ? 3.0e12
                                                  : (mt == 1 ? (gateup ? 6.0e12 : 5.4e12)
                                                             : (gateup ? 5.3e12 : (wp.nw == 16 ? 5.9e12 : 4.9e12)));
  const double walk = passes * (bytes / rate + 5e-6);
  const int ncb = (n_out + (gateup ? 127 : 255)) / (gateup ? 128 : 256);
  const int slices = gateup ? 1 : gg::k_slices_for(est_rows, n_local, ncb, K, exact);
  const double units = (double)gg::expected_tiles(est_rows, n_local, ncb, exact) * slices;
  const double k_slice = (double)K / slices;
  const double panel = 256.0 * k_slice * 2.0;  // bytes of weights one tile streams
  const double mfma_pace = k_slice / 64.0 * 1.3e-6 * fmin(1.0, rows_hi / 256.0);
  const double by_flops = 2.0 * mats * est_rows * (double)n_out * K / 1.2e15;
  double tiled;
  if (gateup) {
    const double by_rounds = fmax(units / 256.0, 1.0) * (fmax(panel / 45e9, mfma_pace) + 8e-6);
    const double by_hbm = units * panel / 5.7e12 + 4e-6;  // all tiles together: their panels at the HBM rate
    tiled = fmax(fmax(by_rounds, by_hbm), by_flops);
  } else {
    const double per_cu = fmin(45e9, 5.4e12 / fmin(units, 256.0));
    tiled = fmax(fmax(units / 256.0, 1.0) * (fmax(panel / per_cu, mfma_pace) + 8e-6), by_flops);
  }
  return walk < tiled;
}

}  // namespace

// Streaming tiles for experts of up to 160 planned rows, 64, 128 or 160 rows high: there the GEMM is bound by HBM, and this kernel streams
// at 5.2-6.0 TB/s where the tiled ones reach 3.3-5.4 and the streaming one 4.0-5.4 (in one pass of 16 rows up to 6.0).
// Measured alone on weights that are not in any cache, us, before / this kernel, gate/up and down projection, by average
// rows per expert: Qwen1.5-MoE (60 experts) 3 rows 119 / 113, 65 / 58; 14: 139 / 127, 86 / 67; 36: 144 / 130, 82 / 74;
// 100: 161 / 144, 96 / 95; Mixtral (8 experts) 3: 278 / 281, 160 / 146; 14: 343 / 317, 185 / 163; 100: 389 / 333, 199 /
// 201; its TP=4 slice 14: 96 / 83, 52 / 45; 100: 104 / 90, 63 / 57; Qwen2-57B (64 experts) 14: 417 / 395, 254 / 208; its
// TP=8 slice (K = 320) 14: 64 / 54, 147 / 32.
// With 160 rows: TP=4 slice of Mixtral, 130 rows 112 / 93, 71 / 64, 145: 115 / 93, 76 / 67; Qwen1.5-MoE 130: 164 / 147, 97 / 98;
// Qwen2-57B TP=2 EP=2 130: 151 / 134, 88 / 87; 8 experts of TP=2, 145: 222 / 180, 130 / 126.  An expert-parallel shard takes
// them by its balanced share: the passes of the experts that got more share their weights in L2.
// Two passes of 160 rows share them, too, at 1.2 us per k-tile of 160 x 256: the down projection just above one 256-row
// block, where the tiled kernels have tall blocks or remainders, (Qwen1.5-MoE 250 rows 143 / 131, 270: 144 / 137, 290: 167 / 140;
// Mixtral TP=2 270: 173 / 136, TP=4 104 / 74, TP=8 59 / 43; Qwen2-57B 270: 406 / 396; 30 experts of Qwen1.5 250: 59 / 65, 270: 73 /
// 66; experts of exactly 256 or 272 rows each, with nothing left over, are 5 % faster tiled, Qwen1.5-MoE 122 / 128), and gate/up projections whose tall tiles leave most of a round idle (estimated; 30 experts of Qwen1.5 270: 124 / 117, its
// TP=2 slice 136 / 118, Mixtral TP=8 99 / 78, Qwen2-57B TP=2 EP=2 201 / 188; not Qwen1.5 214 / 229, Mixtral TP=4 142 / 149).
// Where it does not pay: too few output strips of 16 columns to keep 256 workgroups in tiles (a single expert's down
// projection: Mixtral EP=8 (256 strips) 33 / 67, EP=4 (512) 52 / 73; 1024 strips 94 / 89, but with more than
// 64 rows, where a k-tile's MFMAs want wide tiles, 110 / 169; 1792 strips 50 / 42) or, with 16 rows and fewer, to beat
// the streaming kernel (Qwen2-57B's shared expert under TP=8, 160 strips, 8 rows 14.7 / 19.5; the tiny layer, K = 512, 3 rows
// 6.4 / 7.8).  Tiles of 256 weight rows from 4 gate/up strips per workgroup on (TP=4 slice of Mixtral, 7: 83 / 89 with 128; 8
// experts of TP=8, 2.8: 24 / 22); the down projection's are the same within 2 %.
FlowPlan flow_plan(int cap_rows, int est_rows, int n_local, int n_out, int K, bool gateup) {
  const FlowPlan none = {0, 0};
  if (cap_rows == 0 || K % 64 != 0 || K < 192 || K > (1 << 21) || n_out % 16 != 0) return none;  // (K: 32-bit offsets in a tile)
  const long strips = (long)(est_rows < n_local ? est_rows : n_local) * (n_out / 16);
  const double bytes = (double)strips * 16 * (gateup ? 2 : 1) * K * 2;
  if ((gateup ? strips < 320 : strips < 1024) || bytes < 32e6) return none;
  const double hi = planned_rows_hi(cap_rows, est_rows, n_local), avg = (double)est_rows / n_local;
  if (hi <= 16.0 && (strips < 448 || (gateup && K >= 4096 && bytes > 1e9))) return none;
  if (hi <= 64.0) return FlowPlan{64, gateup && strips >= 1024 ? 256 : 128};
  if (!gateup && strips < 1700) return none;
  // a few large experts of a batch that may be skewed: the popular one's last pass is mostly empty between these averages
  // (Mixtral EP=4 under Zipf(1.2), layer, 200 / 308 tokens 202 / 206 tiled, 208 / 225; 400 and 450: 287 / 300, 254 / 280; smaller
  // weights gain throughout, TP=4 EP=2 308 tokens 156 / 137)
  if (est_rows < cap_rows && n_local < 8 && avg < 100.0 && bytes > (gateup ? 300e6 : 150e6)) return none;
  if (hi <= 128.0) return FlowPlan{128, 256};
  const bool exact = n_local == 1 && est_rows == cap_rows;
  if (avg + (exact ? 0.0 : 2.0 * sqrt(avg)) <= 165.0) return FlowPlan{160, 256};
  if (hi < 283.0 || hi > 326.0 || est_rows < cap_rows) return none;
  if (!gateup) return FlowPlan{160, 256};
  const int nk = K / 64, tall = n_local * ((n_out + 127) / 128);
  const double flow_us = gf::tile_cost(2 * n_local, gf::workgroups(false), n_local, n_out / 16, 160, 256, true, nullptr) * nk * 0.15 + 6.0;
  const double tall_us = (tall + 255) / 256 * (nk * 1.6 + 12.0);
  return flow_us < 0.95 * tall_us ? FlowPlan{160, 256} : none;
}

// The GEMMs of `which` (kTall*) that run the kernel with tall row blocks.
int tall_gemms(int cap_rows, int est_rows, int n_local, int H, int I_s, int which) {
  if (!tall_blocks_allowed(est_rows, n_local, H, I_s)) return 0;
  int out = 0;
  if ((which & kTallGateUp) && expects_tall_blocks(cap_rows, est_rows, n_local, (I_s + 127) / 128, H / gg::BK, false))
    out |= kTallGateUp;
  const int ncb = (H + 255) / 256, nk = I_s / gg::BK;
  if ((which & kTallDown) &&
      expects_tall_blocks(cap_rows, est_rows, n_local, ncb, nk, gg::slice_plan(cap_rows, ncb, I_s).max_slices > 1))
    out |= kTallDown;
  if ((which & kTallDownBf16) && expects_tall_blocks(cap_rows, est_rows, n_local, ncb, nk, false)) out |= kTallDownBf16;
  return out;
}

int tiled_block_rows(int cap_rows, int est_rows, int n_local, int H, int I_s) {
  (void)cap_rows;
  return prefer_even(est_rows, n_local, H, I_s) ? gg::kEvenRows : 256;
}

size_t ffn_workspace_bytes(int cap_rows, int est_rows, int n_local, int H, int I_s) {
  if (cap_rows == 0) return 0;
  // what the tiled kernels need is always covered: MOE_FFN_TILED may overrule the estimate
  const size_t tiled = (size_t)gg::slice_plan(cap_rows, (H + 255) / 256, I_s).scratch_rows * H * sizeof(float);
  if (!prefer_walk(cap_rows, est_rows, n_local, H, I_s, false)) return tiled;
  const gw::WalkPlan p2 = gw::plan_for(I_s, decode_mt(cap_rows, est_rows, n_local), true);
  const int slices = p2.nw == 0 ? 1 : p2.slices;
  const size_t walk = slices > 1 ? (size_t)slices * cap_rows * H * sizeof(float) : 0;
  return walk > tiled ? walk : tiled;
}

void walk_split(int K, int mt, bool down, int32_t out[3]) {
  const gw::WalkPlan p = gw::plan_for(K, mt, down);
  out[0] = p.nw;
  out[1] = p.steps;
  out[2] = p.slices;
}

void ffn_plan(int cap_rows, int est_rows, int n_local, int H, int I_s, int32_t out[4]) {
  const bool walk1 = prefer_walk(cap_rows, est_rows, n_local, I_s, H, true),
             walk2 = prefer_walk(cap_rows, est_rows, n_local, H, I_s, false);
  const int mt = decode_mt(cap_rows, est_rows, n_local);
  out[0] = walk1;
  out[1] = walk2;
  out[2] = mt;
  if (walk2) {
    const gw::WalkPlan p2 = gw::plan_for(I_s, mt, true);
    out[3] = p2.nw == 0 ? 1 : p2.slices;
  } else {
    out[3] = gg::slice_plan(cap_rows, (H + 255) / 256, I_s).max_slices;
  }
}

hipError_t launch_expert_ffn(const void* x_perm, RowMap rows, const int32_t* expert_offsets, int cap_rows, int est_rows,
                             int n_local, int H, int I_s, const void* w_gate, const void* w_up, const void* w_down,
                             void* h_ws, void* y_perm, void* workspace, size_t workspace_bytes, uint32_t flags,
                             int32_t* tickets, hipStream_t stream) {
  (void)workspace_bytes;
  if (cap_rows == 0) return hipSuccess;
  // each GEMM picks its kernel family on its own: h is row-major bf16 for both
  const int mt = decode_mt(cap_rows, est_rows, n_local);
  const bool even = !tall_blocks_allowed(est_rows, n_local, H, I_s) && prefer_even(est_rows, n_local, H, I_s);
  auto run = [&](bool walk, uint32_t f) {
    if (!walk && even)
      return launch_pair_even(x_perm, rows, expert_offsets, cap_rows, n_local, H, I_s, w_gate, w_up, w_down, h_ws,
                              y_perm, f, stream);
    if (!walk)
      return launch_pair_dlds<256>(x_perm, rows, expert_offsets, cap_rows, est_rows, n_local, H, I_s, w_gate, w_up, w_down,
                                   h_ws, y_perm, workspace, f, stream);
    if (mt == 1)
      return launch_pair_decode<1>(x_perm, rows, expert_offsets, cap_rows, n_local, H, I_s, w_gate, w_up, w_down, h_ws,
                                   y_perm, workspace, f, stream);
    return launch_pair_decode<2>(x_perm, rows, expert_offsets, cap_rows, n_local, H, I_s, w_gate, w_up, w_down, h_ws,
                                 y_perm, workspace, f, stream);
  };
  const bool tiled_only = (flags & MOE_FFN_TILED) != 0;
  const bool walk1 = !tiled_only && prefer_walk(cap_rows, est_rows, n_local, I_s, H, true),
             walk2 = !tiled_only && prefer_walk(cap_rows, est_rows, n_local, H, I_s, false);
  const FlowPlan none = {0, 0};
  const FlowPlan flow1 = tiled_only ? none : flow_plan(cap_rows, est_rows, n_local, I_s, H, true),
                 flow2 = tiled_only ? none : flow_plan(cap_rows, est_rows, n_local, H, I_s, false);
  const bool leave_room = (flags & MOE_FFN_LEAVE_ROOM) != 0;
  // the counters pay where another stream holds compute units when the launch starts; alone they cost the longer look-up
  // (TP=4 slice of Qwen1.5, 22 rows per expert, down projection 26 us dealt, 31 from a counter; launches of 100 us the same)
  if (!leave_room) tickets = nullptr;
  if (!(flags & MOE_FFN_SKIP_GATEUP)) {
    const bool both = flow1.rows == 0 && flow2.rows == 0 && walk1 == walk2;
    const hipError_t err =
        flow1.rows != 0 ? launch_flow(flow1, true, true, x_perm, rows, expert_offsets, n_local, w_gate, w_up, I_s,
                                      H, h_ws, tickets, leave_room, stream)
                        : run(walk1, both ? flags : flags | MOE_FFN_SKIP_DOWN);
    if (err != hipSuccess || both) return err;
  }
  if (flags & MOE_FFN_SKIP_DOWN) return hipSuccess;
  if (flow2.rows != 0)
    return launch_flow(flow2, false, (flags & MOE_Y_PERM_BF16) != 0, h_ws, RowMap{nullptr, 1}, expert_offsets,
                       n_local, w_down, nullptr, H, I_s, y_perm, tickets == nullptr ? nullptr : tickets + 1, leave_room,
                       stream);
  return run(walk2, flags | MOE_FFN_SKIP_GATEUP);
}

}  // namespace moe
