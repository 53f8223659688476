// INT4 per-group backup of expert weights: dequantise to bf16 (the step on the paper's strategy
// switching path, "The Dynamic Parallelism Transition Strategy") and quantise (builds the backup).
//
// Both kernels are pure streaming: dequantise reads 0.5625 bytes and writes 2 bytes per weight, so
// the design goal is HBM efficiency.  A lane handles 8 consecutive weights: one 4-byte load of
// codes, one 16-byte store of bf16 (both fully coalesced across the wavefront); the 8 lanes of a
// group share one 4-byte (scale, min) word, which the first of them pulls into the L1.  Four
// independent items per lane keep enough loads in flight.
#include "moe_int4.h"
#include "moe_internal.hpp"

namespace moe {
namespace {

constexpr int kThreads = 256;
constexpr int kItems = 4;                                  // 8-weight items per lane
constexpr int64_t kBlockWeights = (int64_t)kThreads * kItems * 8;  // 8192

__global__ __launch_bounds__(kThreads) void int4_dequantize_kernel(const uint32_t* __restrict__ codes,
                                                                   const uint32_t* __restrict__ qparams,
                                                                   int64_t n_items, uint4* __restrict__ out) {
  const int64_t base = (int64_t)blockIdx.x * (kThreads * kItems) + threadIdx.x;
  uint32_t c[kItems], qp[kItems];
#pragma unroll
  for (int it = 0; it < kItems; ++it) {
    const int64_t i = base + it * kThreads;
    if (i < n_items) {
      c[it] = __builtin_nontemporal_load(codes + i);
      qp[it] = qparams[i >> 3];
    }
  }
#pragma unroll
  for (int it = 0; it < kItems; ++it) {
    const int64_t i = base + it * kThreads;
    if (i < n_items) {
      const float scale = bf16_lo(qp[it]), mn = bf16_hi(qp[it]);
      float v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = fmaf((float)((c[it] >> (4 * j)) & 15u), scale, mn);
      uint4 o;
      o.x = pack_bf16x2(v[0], v[1]);
      o.y = pack_bf16x2(v[2], v[3]);
      o.z = pack_bf16x2(v[4], v[5]);
      o.w = pack_bf16x2(v[6], v[7]);
      __builtin_nontemporal_store(o.x, &out[i].x);
      __builtin_nontemporal_store(o.y, &out[i].y);
      __builtin_nontemporal_store(o.z, &out[i].z);
      __builtin_nontemporal_store(o.w, &out[i].w);
    }
  }
}

// Minimum / maximum in the form the hardware has for three operands (v_minimum3_f32): fminf / fmaxf make the
// compiler quiet each of the loaded values first, one more instruction per weight.  Unlike those they hand a NaN on,
// which is how quantize_block finds a group that has one.
__device__ __forceinline__ float min2(float a, float b) { return __builtin_elementwise_minimum(a, b); }
__device__ __forceinline__ float max2(float a, float b) { return __builtin_elementwise_maximum(a, b); }
template <int CTRL>
__device__ __forceinline__ float dpp_move(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}

// range / 15, correctly rounded: one Newton correction with the rounded 1/15 is exact (Markstein) away from
// overflow and underflow, 3 instructions against the 12 of a general division.
__device__ __forceinline__ float fifteenth(float range) {
  constexpr float kInv = 1.f / 15.f;
  if (range > 1e-30f && range < 1e38f) {
    const float q = range * kInv;
    return fmaf(fmaf(-q, 15.f, range), kInv, q);
  }
  return range / 15.0f;
}

// The eight codes of one lane, packed: rint((w - min) / scale), an IEEE division per weight as it stands, and
// done as such those divisions (about 25 vector instructions per weight) bound the kernel instead of HBM.
// Here the quotient is bracketed by products with the group's reciprocal less and plus 2^-20 of it, rounded to integers
// by adding 1.5 * 2^23; the reciprocal is good to 2^-23, so the fp32 quotient lies in the bracket and where both
// ends give the same integers (one comparison for all eight: no digit of the packed sums can cancel) that
// is the code.  Else a half integer is near, and the remainder decides: r = (w - min) - q * scale is exact in one
// fma (q has 4 bits, scale 8, and |r| is at most scale / 2 and a little), q is the lower end, and the fp32 quotient
// is a half integer only if the exact one is (it cannot round to one: (q + 1/2) has so few bits that its
// neighbours w - min are more than half an ulp of the quotient away).  A few weights in a thousand of bf16 data
// are exact ties, so most wavefronts take that second look, and none of it divides.  A subnormal
// scale, which may be far from range / 15 and has no finite reciprocal, takes the division itself, and so does a
// group with a NaN (whose own code is 0).
__device__ __forceinline__ uint32_t pack_codes(const float (&v)[8], float mn, float scale, bool has_nan) {
  constexpr float kShift = 12582912.f;  // 1.5 * 2^23
  constexpr uint32_t kShiftSum = 0x4B400000u * 0x11111111u;
  uint32_t packed = 0;
  if (has_nan || !(scale >= 1.17549435e-38f && scale < 3e38f)) {
#pragma unroll 1
    for (int j = 0; j < 8; ++j) {
      float q = rintf((v[j] - mn) / scale);
      q = fminf(fmaxf(q, 0.f), 15.f);
      packed |= (uint32_t)q << (4 * j);
    }
    return packed;
  }
  const float inv = __builtin_amdgcn_rcpf(scale);
  const float lo = inv * (1.f - 0x1p-20f), hi = inv * (1.f + 0x1p-20f);
  float d[8], t[8];
  uint32_t upper = 0;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    d[j] = v[j] - mn;
    t[j] = fmaf(d[j], lo, kShift);
    packed += __float_as_uint(t[j]) << (4 * j);
    upper += __float_as_uint(fmaf(d[j], hi, kShift)) << (4 * j);
  }
  if (packed != upper) {
    const float half = 0.5f * scale;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const float r = fmaf(-(t[j] - kShift), scale, d[j]);
      const uint32_t odd = __float_as_uint(t[j]) & 1u;
      packed += (uint32_t)(r > half || (r == half && odd != 0)) << (4 * j);
    }
  }
  return packed - kShiftSum;
}

// 8 lanes per group: each loads 8 weights (16 bytes), min / max meet by three cross-lane steps inside
// the eight lanes (data-parallel primitives, no trip through the LDS crossbar).  Four independent items per
// lane, all loads first, as in the dequantise kernel.  352 M weights (902 MB): 222 us (4.1 TB/s) with a division per
// weight, 178 us with a remainder check that sent exact ties to the division, 142 us (6.34 TB/s, HBM) now.
// FULL: every item of the block exists, so the loads carry no branches and each item waits for its own only.
template <bool FULL>
__device__ __forceinline__ void quantize_block(const uint4* __restrict__ w, int64_t base, int64_t n_items,
                                               uint32_t* __restrict__ codes, uint32_t* __restrict__ qparams) {
  // n_items is a multiple of 8, so the 8 lanes of a group are in range together
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  u32x4 raw[kItems];
#pragma unroll
  for (int it = 0; it < kItems; ++it) {
    const int64_t i = base + it * kThreads;
    if (FULL || i < n_items) raw[it] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(w) + i);
    else raw[it] = u32x4{0, 0, 0, 0};
  }
#pragma unroll
  for (int it = 0; it < kItems; ++it) {
    const int64_t i = base + it * kThreads;
    const u32x4 q = raw[it];
    const float v[8] = {bf16_lo(q.x), bf16_hi(q.x), bf16_lo(q.y), bf16_hi(q.y),
                        bf16_lo(q.z), bf16_hi(q.z), bf16_lo(q.w), bf16_hi(q.w)};
    float mn = v[0], mx = v[0];
#pragma unroll
    for (int j = 1; j < 8; ++j) {
      mn = min2(mn, v[j]);
      mx = max2(mx, v[j]);
    }
    // lanes 1 and 2 apart, then mirrored within the eight (each quad already agrees)
    mn = min2(mn, dpp_move<0xB1>(mn));
    mx = max2(mx, dpp_move<0xB1>(mx));
    mn = min2(mn, dpp_move<0x4E>(mn));
    mx = max2(mx, dpp_move<0x4E>(mx));
    mn = min2(mn, dpp_move<0x141>(mn));
    mx = max2(mx, dpp_move<0x141>(mx));
    // a NaN in the group: the extremes of its other weights, so that one bad weight costs no more than its own value
    const bool has_nan = mn != mn;
    if (has_nan) {
      mn = mx = v[0];
#pragma unroll
      for (int j = 1; j < 8; ++j) {
        mn = fminf(mn, v[j]);
        mx = fmaxf(mx, v[j]);
      }
#pragma unroll
      for (int o = 1; o < 8; o <<= 1) {  // the eight lanes of a group are here together
        mn = fminf(mn, __shfl_xor(mn, o, kWave));
        mx = fmaxf(mx, __shfl_xor(mx, o, kWave));
      }
    }
    const uint32_t scale_bits = f32_to_bf16_bits(fifteenth(mx - mn));
    const float scale = bf16_bits_to_f32(scale_bits);
    const uint32_t packed = scale > 0.f ? pack_codes(v, mn, scale, has_nan) : 0u;
    if (FULL || i < n_items) {
      __builtin_nontemporal_store(packed, codes + i);
      if ((i & 7) == 0) qparams[i >> 3] = scale_bits | (__float_as_uint(mn) & 0xFFFF0000u);  // mn is a bf16 value
    }
  }
}

__global__ __launch_bounds__(kThreads) void int4_quantize_kernel(const uint4* __restrict__ w, int64_t n_items,
                                                                 uint32_t* __restrict__ codes,
                                                                 uint32_t* __restrict__ qparams) {
  const int64_t first = (int64_t)blockIdx.x * (kThreads * kItems);
  if (first + kThreads * kItems <= n_items)
    quantize_block<true>(w, first + threadIdx.x, n_items, codes, qparams);
  else
    quantize_block<false>(w, first + threadIdx.x, n_items, codes, qparams);
}

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

}  // namespace
}  // namespace moe

extern "C" {

int moe_int4_dequantize(const void* codes, const void* qparams, int64_t n_elems, void* w_bf16, void* stream) {
  using namespace moe;
  if (n_elems < 0 || n_elems % MOE_INT4_GROUP != 0) return MOE_ERR_INVALID_ARG;
  if (codes == nullptr || qparams == nullptr || w_bf16 == nullptr) return MOE_ERR_INVALID_ARG;
  if (!aligned16(codes) || !aligned16(qparams) || !aligned16(w_bf16)) return MOE_ERR_INVALID_ARG;
  if (n_elems / kBlockWeights >= 0x7FFFFFFF) return MOE_ERR_UNSUPPORTED_SHAPE;
  if (n_elems == 0) return MOE_OK;
  const int64_t n_items = n_elems / 8;
  const unsigned grid = (unsigned)((n_elems + kBlockWeights - 1) / kBlockWeights);
  hipLaunchKernelGGL(int4_dequantize_kernel, dim3(grid), dim3(kThreads), 0, static_cast<hipStream_t>(stream),
                     static_cast<const uint32_t*>(codes), static_cast<const uint32_t*>(qparams), n_items,
                     static_cast<uint4*>(w_bf16));
  return hipGetLastError() == hipSuccess ? MOE_OK : MOE_ERR_HIP;
}

int moe_int4_quantize(const void* w_bf16, int64_t n_elems, void* codes, void* qparams, void* stream) {
  using namespace moe;
  if (n_elems < 0 || n_elems % MOE_INT4_GROUP != 0) return MOE_ERR_INVALID_ARG;
  if (codes == nullptr || qparams == nullptr || w_bf16 == nullptr) return MOE_ERR_INVALID_ARG;
  if (!aligned16(codes) || !aligned16(qparams) || !aligned16(w_bf16)) return MOE_ERR_INVALID_ARG;
  const int64_t n_items = n_elems / 8;
  // (a bound in blocks of one item per lane, which a grid of blocks of kItems would not need)
  if ((n_items + kThreads - 1) / kThreads >= 0x7FFFFFFF) return MOE_ERR_UNSUPPORTED_SHAPE;
  if (n_elems == 0) return MOE_OK;
  const unsigned grid = (unsigned)((n_elems + kBlockWeights - 1) / kBlockWeights);
  hipLaunchKernelGGL(int4_quantize_kernel, dim3(grid), dim3(kThreads), 0, static_cast<hipStream_t>(stream),
                     static_cast<const uint4*>(w_bf16), n_items, static_cast<uint32_t*>(codes),
                     static_cast<uint32_t*>(qparams));
  return hipGetLastError() == hipSuccess ? MOE_OK : MOE_ERR_HIP;
}

}  // extern "C"
