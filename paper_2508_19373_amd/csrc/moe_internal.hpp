// Internal declarations shared by the HIP translation units of libmoe_shard (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "moe_shard.h"

namespace moe {

constexpr int kWave = 64;

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

// bf16 bit pattern <-> fp32
__device__ __forceinline__ float bf16_bits_to_f32(uint32_t bits16) { return __uint_as_float(bits16 << 16); }
__device__ __forceinline__ float bf16_lo(uint32_t packed) { return __uint_as_float(packed << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t packed) { return __uint_as_float(packed & 0xFFFF0000u); }

// fp32 -> bf16, round to nearest even, by the hardware converter (v_cvt_pk_bf16_f32)
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  const f32x2_t v = {lo, hi};
  const bf16x2_t b = __builtin_convertvector(v, bf16x2_t);
  return *reinterpret_cast<const uint32_t*>(&b);
}
__device__ __forceinline__ uint32_t f32_to_bf16_bits(float f) { return pack_bf16x2(f, 0.f) & 0xFFFFu; }

// Reduction over the 64 lanes, every lane gets it: lanes 32, 16, 8, 4, 2 and 1 apart in this order.  Row swaps and
// data-parallel moves, a few cycles each where a shuffle is a trip through the LDS crossbar.  (4 apart by a rotation
// within 16 lanes: the values repeat every 8 lanes there.)
template <typename Op>
__device__ __forceinline__ float wave_reduce(float v, Op op) {
#ifdef __HIP_DEVICE_COMPILE__
  const auto half = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = op(__uint_as_float(half[0]), __uint_as_float(half[1]));
  const auto row = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = op(__uint_as_float(row[0]), __uint_as_float(row[1]));
  const auto move = [](float x, auto ctrl) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), decltype(ctrl)::value, 0xF, 0xF, true));
  };
  v = op(v, move(v, std::integral_constant<int, 0x128>{}));  // row_ror:8
  v = op(v, move(v, std::integral_constant<int, 0x124>{}));  // row_ror:4
  v = op(v, move(v, std::integral_constant<int, 0x4E>{}));   // quad_perm 2,3,0,1
  v = op(v, move(v, std::integral_constant<int, 0xB1>{}));   // quad_perm 1,0,3,2
#endif
  return v;
}
__device__ __forceinline__ float wave_sum(float v) {
  return wave_reduce(v, [](float a, float b) { return a + b; });
}
__device__ __forceinline__ float wave_max(float v) {
  return wave_reduce(v, [](float a, float b) { return fmaxf(a, b); });
}

// Where the rows of the first GEMM come from: row r of the input is x[row_src[r] / k] (the token of
// assignment row_src[r]); row_src == nullptr means the input is already permuted (row r itself).
struct RowMap {
  const int32_t* row_src;
  int k;
  __host__ __device__ inline int operator()(int r) const { return row_src ? row_src[r] / k : r; }
};

// launchers (each returns hipGetLastError() after enqueueing on `stream`)
hipError_t launch_route_topk(const void* x, const float* w_router, float* logits, int T, int H, int E, int k,
                             uint32_t flags, int32_t* topk_idx, float* topk_w, hipStream_t stream);
// Whether launch_route_topk of such a call computes the logits in a kernel of their own, and that kernel alone.
bool route_has_logits_kernel(int T, int H, int E, uint32_t flags);
hipError_t launch_route_logits(const void* x, const float* w_router, float* logits, int T, int H, int E, hipStream_t stream);
hipError_t launch_permute(const void* x, const int32_t* topk_idx, int T, int k, int H, int n_local, int offset,
                          void* x_perm, int32_t* expert_offsets, int32_t* row_src, int32_t* slot_row,
                          void* workspace, hipStream_t stream, int32_t* tickets = nullptr);
size_t permute_workspace_bytes(int T, int k, int n_local);
// launch_route_topk and launch_permute of a small batch whose logits are given (or already computed), in one kernel:
// whether it takes them (nothing is enqueued if not).
bool route_permute_fits(int T);
hipError_t launch_route_permute(const float* logits, int T, int E, int k, uint32_t flags, int32_t* topk_idx, float* topk_w,
                                const void* x, int H, int n_local, int offset, void* x_perm, int32_t* expert_offsets,
                                int32_t* row_src, int32_t* slot_row, hipStream_t stream, int32_t* tickets);
// Words at the end of that workspace for launch_permute to clear as `tickets` (kTickets of them, nullptr: none): the counters the GEMM
// kernels of the same forward take their tiles from.
constexpr int kTickets = 2;
int32_t* permute_tickets(void* workspace, int T, int k, int n_local);
// The same with the library's own static scratch; permute_static_counts: int32 counts it would use.
hipError_t launch_permute_static(const void* x, const int32_t* topk_idx, int T, int k, int H, int n_local, int offset,
                                 void* x_perm, int32_t* expert_offsets, int32_t* row_src, int32_t* slot_row,
                                 hipStream_t stream);
size_t permute_static_counts(int T, int k, int n_local);
// est_rows: the rows this shard expects (cap_rows scaled by its share of the experts); it steers the
// choice of kernels and K slices only, every bound is taken from cap_rows.
hipError_t launch_expert_ffn(const void* x_perm, RowMap rows, const int32_t* expert_offsets, int cap_rows, int est_rows,
                             int n_local, int H, int I_s, const void* w_gate, const void* w_up, const void* w_down,
                             void* h_ws, void* y_perm, void* workspace, size_t workspace_bytes, uint32_t flags,
                             int32_t* tickets, hipStream_t stream);
size_t ffn_workspace_bytes(int cap_rows, int est_rows, int n_local, int H, int I_s);
// What launch_expert_ffn would do: {GEMM1 by the walk kernel, GEMM2 by the walk kernel, rows per
// walk pass / 16, K slices of GEMM2}.
void ffn_plan(int cap_rows, int est_rows, int n_local, int H, int I_s, int32_t out[4]);
// How the walk kernel would cut K with 16 * mt rows per pass: wavefronts (0: not instantiated, the generic streaming kernel runs),
// k32 steps per wavefront, slices.
void walk_split(int K, int mt, bool down, int32_t out[3]);
// Row-block height of the tiled kernels for such a call (256, or 160 for the one-height work list).
int tiled_block_rows(int cap_rows, int est_rows, int n_local, int H, int I_s);
// Which GEMMs of such a call, when tiled, run the kernel whose full row blocks may take their expert's remainder: those
// of `which`, MOE_DEBUG_TALL_*.
constexpr int kTallGateUp = 1, kTallDown = 2, kTallDownBf16 = 4;
int tall_gemms(int cap_rows, int est_rows, int n_local, int H, int I_s, int which);
int expected_rows(int cap_rows, const moe_shard_t* shard);
// The streaming tiles (grouped_flow.hpp): rows and weight rows of its tiles for one of
// the two GEMMs of such a call, rows = 0 where another kernel runs it.
struct FlowPlan {
  int rows, cols;
};
FlowPlan flow_plan(int cap_rows, int est_rows, int n_local, int n_out, int K, bool gateup);
// ticket: a zero in device memory (nullptr: tiles are dealt in turn)
hipError_t launch_flow(const FlowPlan& plan, bool gateup, bool out_bf16, const void* A, RowMap rows,
                       const int32_t* expert_offsets, int n_local, const void* B0, const void* B1,
                       int n_out, int K, void* C, int32_t* ticket, bool leave_room, hipStream_t stream);
hipError_t launch_combine(const void* y_perm, const int32_t* slot_row, const float* topk_w, int T, int k, int H,
                          const void* y_shared, const void* x, const float* w_shared_gate, void* y_out,
                          bool y_perm_bf16, bool out_f32, hipStream_t stream);

}  // namespace moe
