// Top-K selection and gate weights of one token by one wavefront (paper, "MoE Model Architectures").
#pragma once
#include "moe_internal.hpp"

namespace moe {

// myl[s] holds the logit of expert lane + 64*s (-inf past E).  k rounds of a wave-wide maximum on (logit desc, expert id
// asc), then softmax over all E logits evaluated at the selected ones.  Bound by the chain of cross-lane steps: the maximum
// takes six register moves and the lowest lane that holds it one ballot (60 experts, k = 4, 32 tokens: the kernel 10.2 us with
// shuffled (logit, id) pairs, 4.5 now; a launch of any kind takes 4).  A token whose remaining logits are all NaN (outside
// the contract) gets its lowest remaining experts.
template <int EPL>
__device__ __forceinline__ void select_topk(const float (&myl)[EPL], int lane, int E, int k, uint32_t flags,
                                            int32_t* __restrict__ idx_out, float* __restrict__ w_out,
                                            int32_t* idx_lds = nullptr) {
  uint32_t taken = 0;  // bit s set: this lane's slot s already selected
  float sel_v = 0.f;
  int sel_i = 0;
  float vmax = 0.f;
  for (int j = 0; j < k; ++j) {
    float bv = -INFINITY;
#pragma unroll
    for (int s = 0; s < EPL; ++s)
      if (lane + s * kWave < E && !(taken & (1u << s))) bv = fmaxf(bv, myl[s]);
    bv = wave_max(bv);
    int bi = -1, first = -1;
#pragma unroll
    for (int s = EPL - 1; s >= 0; --s) {  // the lowest id last
      const bool open = lane + s * kWave < E && !(taken & (1u << s));
      const unsigned long long any = __ballot(open), hit = __ballot(open && myl[s] == bv);
      if (any != 0) first = s * kWave + __ffsll((long long)any) - 1;
      if (hit != 0) bi = s * kWave + __ffsll((long long)hit) - 1;
    }
    if (bi < 0) bi = first;
    if ((bi & 63) == lane) taken |= 1u << (bi >> 6);
    if (j == 0) vmax = bv;
    if (lane == j) {
      sel_v = bv;
      sel_i = bi;
    }
  }
  // softmax denominator over all E experts (max logit is the first selected one)
  float part = 0.f;
#pragma unroll
  for (int s = 0; s < EPL; ++s) {
    const int e = lane + s * kWave;
    if (e < E) part += expf(myl[s] - vmax);
  }
  const float denom_all = wave_sum(part);
  const float num = (lane < k) ? expf(sel_v - vmax) : 0.f;
  const float denom_sel = wave_sum(num);
  if (lane < k) {
    idx_out[lane] = sel_i;
    if (idx_lds != nullptr) idx_lds[lane] = sel_i;
    w_out[lane] = num / ((flags & MOE_RENORM_TOPK) ? denom_sel : denom_all);
  }
}

}  // namespace moe
