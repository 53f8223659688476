// Launches of the streaming tiles (grouped_flow.hpp); flow_plan in expert_ffn.hip says when they run.
#include "grouped_flow.hpp"

namespace moe {
namespace {

template <int BM, int BN, bool GATEUP, typename OutT>
hipError_t launch(const uint16_t* A, RowMap rows, const int32_t* expert_offsets, int n_local,
                  const uint16_t* B0, const uint16_t* B1, int n_out, int K, void* C, int32_t* ticket, bool leave_room,
                  hipStream_t stream) {
  const int regions = gf::k_regions(n_local, BM);
  hipLaunchKernelGGL((gf::grouped_flow_kernel<BM, BN, GATEUP, OutT>), dim3(gf::workgroups(leave_room)), dim3(gf::kThreads), 0, stream, A,
                     expert_offsets, n_local, regions, gf::k_step(n_local, regions, K / gf::BK), B0, B1, n_out, K, static_cast<OutT*>(C), rows, ticket);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_flow(const FlowPlan& plan, bool gateup, bool out_bf16, const void* A, RowMap rows,
                       const int32_t* expert_offsets, int n_local, const void* B0, const void* B1,
                       int n_out, int K, void* C, int32_t* ticket, bool leave_room, hipStream_t stream) {
  const uint16_t *a = static_cast<const uint16_t*>(A), *b0 = static_cast<const uint16_t*>(B0),
                 *b1 = static_cast<const uint16_t*>(B1);
#define MOE_FLOW(BM, BN, GATEUP, OutT) \
  return launch<BM, BN, GATEUP, OutT>(a, rows, expert_offsets, n_local, b0, b1, n_out, K, C, ticket, leave_room, stream)
  if (gateup) {
    if (plan.rows == 160) MOE_FLOW(160, 256, true, uint16_t);
    if (plan.rows == 128) MOE_FLOW(128, 256, true, uint16_t);
    if (plan.cols == 256) MOE_FLOW(64, 256, true, uint16_t);
    MOE_FLOW(64, 128, true, uint16_t);
  }
  if (out_bf16) {
    if (plan.rows == 160) MOE_FLOW(160, 256, false, uint16_t);
    if (plan.rows == 128) MOE_FLOW(128, 256, false, uint16_t);
    MOE_FLOW(64, 128, false, uint16_t);
  }
  if (plan.rows == 160) MOE_FLOW(160, 256, false, float);
  if (plan.rows == 128) MOE_FLOW(128, 256, false, float);
  MOE_FLOW(64, 128, false, float);
#undef MOE_FLOW
}

}  // namespace moe
