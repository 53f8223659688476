// Weighted un-permute / combine of the Top-K expert outputs (paper, "MoE Model Architectures":
// each token's result is the gate-weighted mix of its selected experts), plus the always-active
// shared expert scaled by sigmoid(x . w_s).
//
// Token-major gather: one workgroup per token walks the token's k slots in order and sums in
// fp32, so every output row is written exactly once, coalesced, with no atomics -- the result
// is deterministic.  HBM-bound: reads k rows of y_perm, writes one row of y.
#include "moe_internal.hpp"

namespace moe {
namespace {

constexpr int kCombThreads = 256;

__device__ __forceinline__ void load8(const float* p, float (&v)[8]) {
  const float4 a = *reinterpret_cast<const float4*>(p);
  const float4 b = *reinterpret_cast<const float4*>(p + 4);
  v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
  v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}
__device__ __forceinline__ void load8(const uint16_t* p, float (&v)[8]) {
  const uint4 a = *reinterpret_cast<const uint4*>(p);
  v[0] = bf16_lo(a.x); v[1] = bf16_hi(a.x); v[2] = bf16_lo(a.y); v[3] = bf16_hi(a.y);
  v[4] = bf16_lo(a.z); v[5] = bf16_hi(a.z); v[6] = bf16_lo(a.w); v[7] = bf16_hi(a.w);
}
__device__ __forceinline__ float4 load4(const float* p) { return *reinterpret_cast<const float4*>(p); }
__device__ __forceinline__ float4 load4(const uint16_t* p) {
  const uint2 a = *reinterpret_cast<const uint2*>(p);
  return make_float4(bf16_lo(a.x), bf16_hi(a.x), bf16_lo(a.y), bf16_hi(a.y));
}
__device__ __forceinline__ void store4(float* p, const float4& v) { *reinterpret_cast<float4*>(p) = v; }
__device__ __forceinline__ void store4(uint16_t* p, const float4& v) {
  uint2 o;
  o.x = pack_bf16x2(v.x, v.y);
  o.y = pack_bf16x2(v.z, v.w);
  *reinterpret_cast<uint2*>(p) = o;
}
__device__ __forceinline__ void fma4(float4& acc, float w, const float4& v) {
  acc.x = fmaf(w, v.x, acc.x);
  acc.y = fmaf(w, v.y, acc.y);
  acc.z = fmaf(w, v.z, acc.z);
  acc.w = fmaf(w, v.w, acc.w);
}

// A lane takes 4 columns at a time (whole 1 KB per wavefront and row), kPass of them 1024 columns apart, and loads those of
// kRows rows before it adds the first, so that a token is a memory latency or two and not one per row.  Lane j of every
// wavefront holds slot j's row and weight.  The shared expert's gate is summed while the first rows are on their way.
constexpr int kCols = 4, kPass = 2;
template <typename YT, typename OT, int kRows>
__global__ __launch_bounds__(kCombThreads) void combine_kernel(const YT* __restrict__ y_perm,
                                                              const int32_t* __restrict__ slot_row,
                                                              const float* __restrict__ topk_w, int T, int k, int H,
                                                              const YT* __restrict__ y_shared,
                                                              const uint16_t* __restrict__ x,
                                                              const float* __restrict__ w_shared_gate,
                                                              OT* __restrict__ y_out) {
  __shared__ float red[2][kCombThreads / kWave];
  const int tid = threadIdx.x;
  const bool gated = y_shared != nullptr && w_shared_gate != nullptr;
  int flip = 0;
  for (int t = blockIdx.x; t < T; t += gridDim.x) {
    const int slot = min(tid & (kWave - 1), k - 1);
    const int my_row = slot_row[(size_t)t * k + slot];
    const float my_weight = topk_w[(size_t)t * k + slot];
    auto row_of = [&](int j) { return __builtin_amdgcn_readlane(my_row, j); };
    float gate = 1.f;
    for (int h0 = tid * kCols; h0 < H || h0 == tid * kCols; h0 += kCombThreads * kCols * kPass) {
      float4 v[kRows][kPass], sh[kPass], acc[kPass];
      auto load_rows = [&](int j0) {
#pragma unroll
        for (int j = 0; j < kRows; ++j) {
          const int r = j0 + j < k ? row_of(j0 + j) : -1;
          if (r >= 0) {
#pragma unroll
            for (int p = 0; p < kPass; ++p) {
              const int h = h0 + p * kCombThreads * kCols;
              if (h < H) v[j][p] = load4(y_perm + (size_t)r * H + h);
            }
          }
        }
      };
      load_rows(0);
      if (y_shared != nullptr) {
#pragma unroll
        for (int p = 0; p < kPass; ++p) {
          const int h = h0 + p * kCombThreads * kCols;
          if (h < H) sh[p] = load4(y_shared + (size_t)t * H + h);
        }
      }
      if (gated && h0 == tid * kCols) {  // (every lane comes here once per token)
        float part = 0.f;
        for (int c = tid * 8; c < H; c += kCombThreads * 8) {
          float xv[8], wv[8];
          load8(x + (size_t)t * H + c, xv);
          load8(w_shared_gate + c, wv);
#pragma unroll
          for (int i = 0; i < 8; ++i) part = fmaf(xv[i], wv[i], part);
        }
        part = wave_sum(part);
        if ((tid & (kWave - 1)) == 0) red[flip][tid >> 6] = part;
        __syncthreads();
        float z = 0.f;
#pragma unroll
        for (int w = 0; w < kCombThreads / kWave; ++w) z += red[flip][w];
        flip ^= 1;  // the next token's sums go elsewhere: one barrier per token
        gate = 1.f / (1.f + expf(-z));
      }
#pragma unroll
      for (int p = 0; p < kPass; ++p) acc[p] = make_float4(0.f, 0.f, 0.f, 0.f);
      for (int j0 = 0; j0 < k; j0 += kRows) {
        if (j0 > 0) load_rows(j0);
#pragma unroll
        for (int j = 0; j < kRows; ++j) {
          if (j0 + j < k && row_of(j0 + j) >= 0) {
            const float w = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(my_weight), j0 + j));
#pragma unroll
            for (int p = 0; p < kPass; ++p) fma4(acc[p], w, v[j][p]);
          }
        }
      }
#pragma unroll
      for (int p = 0; p < kPass; ++p) {
        const int h = h0 + p * kCombThreads * kCols;
        if (h < H) {
          if (y_shared != nullptr) fma4(acc[p], gate, sh[p]);
          store4(y_out + (size_t)t * H + h, acc[p]);
        }
      }
    }
  }
}

template <typename YT, typename OT>
hipError_t launch_typed(const void* y_perm, const int32_t* slot_row, const float* topk_w, int T, int k, int H,
                        const void* y_shared, const void* x, const float* w_shared_gate, void* y_out,
                        hipStream_t stream) {
  const int grid = T < 16384 ? T : 16384;
  const auto kernel =
      k <= 2 ? combine_kernel<YT, OT, 2> : (k <= 4 ? combine_kernel<YT, OT, 4> : combine_kernel<YT, OT, 8>);
  hipLaunchKernelGGL(kernel, dim3(grid), dim3(kCombThreads), 0, stream,
                     static_cast<const YT*>(y_perm), slot_row, topk_w, T, k, H, static_cast<const YT*>(y_shared),
                     static_cast<const uint16_t*>(x), w_shared_gate, static_cast<OT*>(y_out));
  return hipGetLastError();
}

}  // namespace

hipError_t launch_combine(const void* y_perm, const int32_t* slot_row, const float* topk_w, int T, int k, int H,
                          const void* y_shared, const void* x, const float* w_shared_gate, void* y_out,
                          bool y_perm_bf16, bool out_f32, hipStream_t stream) {
  if (T == 0) return hipSuccess;
  if (y_perm_bf16) {
    return out_f32 ? launch_typed<uint16_t, float>(y_perm, slot_row, topk_w, T, k, H, y_shared, x, w_shared_gate,
                                                   y_out, stream)
                   : launch_typed<uint16_t, uint16_t>(y_perm, slot_row, topk_w, T, k, H, y_shared, x, w_shared_gate,
                                                      y_out, stream);
  }
  return out_f32
             ? launch_typed<float, float>(y_perm, slot_row, topk_w, T, k, H, y_shared, x, w_shared_gate, y_out, stream)
             : launch_typed<float, uint16_t>(y_perm, slot_row, topk_w, T, k, H, y_shared, x, w_shared_gate, y_out,
                                             stream);
}

}  // namespace moe
