// Token permutation by expert: the dispatch step of the Top-K mechanism (paper, "MoE Model
// Architectures"), restricted to the contiguous expert subset an expert-parallel shard holds
// ("Expert Parallelism").  A stable counting sort of assignment ids a = t*k + j by expert id.
//
// Index kernel for small batches: one 1024-thread workgroup (permute_small).  Ranks among equal experts come from ballots and
// popcounts inside a wavefront, across wavefronts from prefixes in LDS -- no order-dependent atomics, so the result is the
// unique stable order and is identical from run to run.
// Gather kernel: coalesced 16-byte-per-lane row copies x[row_src[r] / k] -> x_perm[r].
#include "moe_internal.hpp"
#include "select_topk.hpp"
#include "unit_list_wave.hpp"

#include <mutex>

namespace moe {
namespace {

// Scratch of moe_permute_static: the per-workgroup expert counts of the large-batch path, in device
// memory that belongs to the library (each GPU the library runs on holds its own copy until the
// process ends).  The name below is a host-side handle only; host code uses the address that
// static_scratch() resolves per device.
constexpr size_t kStaticScratchInts = MOE_PERMUTE_STATIC_MAX_COUNTS;  // 1 MiB
static __device__ __align__(256) int32_t scratch[kStaticScratchInts];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
int32_t* g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on the current device, resolved once per device.
hipError_t static_scratch(int32_t** out) {
  int dev = -1;
  hipError_t err = hipGetDevice(&dev);
  if (err != hipSuccess) return err;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (g_scratch_ptr[dev] == nullptr) {
    void* p = nullptr;
    err = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (err != hipSuccess) return err;
    if (p == nullptr) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = static_cast<int32_t*>(p);
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

constexpr int kIdxThreads = 1024;
constexpr int kIdxWaves = kIdxThreads / kWave;

// Rank of this lane among the lanes of its wavefront with the same expert (ids below 256, -1: none), and how many there
// are: a ballot per bit of the id, whatever the number of experts.
__device__ __forceinline__ int match_rank(int e, int lane, int bits, int& count) {
  unsigned long long same = __ballot(e >= 0);
  for (int b = 0; b < bits; ++b) {
    const unsigned long long set = __ballot((e >> b) & 1);
    same &= ((e >> b) & 1) ? set : ~set;
  }
  count = __popcll(same);
  return __popcll(same & ((1ull << lane) - 1ull));
}
__device__ __forceinline__ int id_bits(int n_local) { return n_local <= 1 ? 0 : 32 - __clz(n_local - 1); }

// Small batches (at most two assignments a thread): each of up to 32 groups of 64 assignments, in order, is ranked by
// one wavefront, which leaves its count of every expert in LDS; a thread per expert adds those up in order, one
// wavefront scans the experts.  expert_of(a): the global expert of assignment a.
template <typename F>
__device__ __forceinline__ void permute_small(F expert_of, int A, int n_local, int offset, int32_t* __restrict__ expert_offsets,
                                              int32_t* __restrict__ row_src, int32_t* __restrict__ slot_row,
                                              const uint4* __restrict__ x, int k, int chunks_per_row,
                                              uint4* __restrict__ x_perm) {
  __shared__ int32_t base[MOE_MAX_EXPERTS];                      // first row of each expert
  __shared__ int32_t group_cnt[2 * kIdxWaves][MOE_MAX_EXPERTS];  // per-group counts, then rows before the group
  __shared__ int32_t total_rows;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid >> 6;
  const int groups = A > kIdxThreads ? 2 * kIdxWaves : kIdxWaves, bits = id_bits(n_local);
  int e[2], rank[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int a = h * kIdxThreads + tid;
    e[h] = a < A ? expert_of(a) - offset : -1;
    if (e[h] < 0 || e[h] >= n_local) e[h] = -1;
  }
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int g = h * kIdxWaves + wv;
    if (g < groups) {
      for (int ee = lane; ee < n_local; ee += kWave) group_cnt[g][ee] = 0;
      int count;
      rank[h] = match_rank(e[h], lane, bits, count);
      if (e[h] >= 0 && rank[h] == 0) group_cnt[g][e[h]] = count;
    }
  }
  __syncthreads();
  for (int ee = tid; ee < n_local; ee += kIdxThreads) {
    int run = 0;
#pragma unroll 8
    for (int g = 0; g < groups; ++g) {
      const int c = group_cnt[g][ee];
      group_cnt[g][ee] = run;
      run += c;
    }
    base[ee] = run;
  }
  __syncthreads();
  if (wv == 0) {  // exclusive scan of up to 256 counts by one wavefront, 64 at a time
    int carry = 0;
    for (int e0 = 0; e0 < n_local; e0 += kWave) {
      const int ee = e0 + lane;
      const int c = (ee < n_local) ? base[ee] : 0;
      const int incl = gg::wave_incl_scan(c);
      if (ee < n_local) {
        base[ee] = carry + incl - c;
        expert_offsets[ee] = carry + incl - c;
      }
      carry += __builtin_amdgcn_readlane(incl, kWave - 1);
    }
    if (lane == 0) expert_offsets[n_local] = total_rows = carry;
  }
  __syncthreads();
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int a = h * kIdxThreads + tid;
    if (a < A) {
      const int row = e[h] >= 0 ? base[e[h]] + group_cnt[h * kIdxWaves + wv][e[h]] + rank[h] : -1;
      slot_row[a] = row;
      if (row >= 0) row_src[row] = a;
    }
  }
  // decode-sized batches: the same workgroup also gathers the rows (x != nullptr), saving a launch
  if (x != nullptr) {
    __syncthreads();
    const int total = total_rows * chunks_per_row;
    for (int i = tid; i < total; i += kIdxThreads) {
      const int r = i / chunks_per_row, c = i - r * chunks_per_row;
      x_perm[(size_t)r * chunks_per_row + c] = x[(size_t)(row_src[r] / k) * chunks_per_row + c];
    }
  }
}

__global__ __launch_bounds__(kIdxThreads) void permute_index_kernel(const int32_t* __restrict__ topk_idx, int A,
                                                                   int n_local, int offset,
                                                                   int32_t* __restrict__ expert_offsets,
                                                                   int32_t* __restrict__ row_src,
                                                                   int32_t* __restrict__ slot_row,
                                                                   const uint4* __restrict__ x, int k,
                                                                   int chunks_per_row, uint4* __restrict__ x_perm,
                                                                   int32_t* __restrict__ tickets) {
  if (tickets != nullptr && threadIdx.x < kTickets) tickets[threadIdx.x] = 0;
  permute_small([=](int a) { return topk_idx[a]; }, A, n_local, offset, expert_offsets, row_src, slot_row, x, k,
                chunks_per_row, x_perm);
}

// Top-K selection and permutation of up to 32 tokens in one workgroup: a wavefront selects for every sixteenth token
// (all of its logits loaded first), the permutation reads the selected experts from LDS.  Two launches of 4 to 5 us each
// become one of 5 (16 tokens, 60 experts, k = 4) to 8 (32, beside another stream); a wavefront takes over 1 us per
// token, so with 128 tokens the one workgroup takes 19 where the two launches take 9.
constexpr int kFusedTokens = 32, kFusedPerWave = kFusedTokens / kIdxWaves;
template <int EPL>
__global__ __launch_bounds__(kIdxThreads) void route_permute_kernel(const float* __restrict__ logits, int T, int E, int k,
                                                                   uint32_t flags, int32_t* __restrict__ topk_idx,
                                                                   float* __restrict__ topk_w, int n_local, int offset,
                                                                   int32_t* __restrict__ expert_offsets,
                                                                   int32_t* __restrict__ row_src,
                                                                   int32_t* __restrict__ slot_row,
                                                                   const uint4* __restrict__ x, int chunks_per_row,
                                                                   uint4* __restrict__ x_perm,
                                                                   int32_t* __restrict__ tickets) {
  __shared__ int32_t s_idx[kFusedTokens * MOE_MAX_TOPK];
  if (tickets != nullptr && threadIdx.x < kTickets) tickets[threadIdx.x] = 0;
  const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x >> 6;
  float myl[kFusedPerWave][EPL];
#pragma unroll
  for (int i = 0; i < kFusedPerWave; ++i) {
    const int t = i * kIdxWaves + wv;
#pragma unroll
    for (int s = 0; s < EPL; ++s) {
      const int e = lane + s * kWave;
      myl[i][s] = t < T && e < E ? logits[(size_t)t * E + e] : -INFINITY;
    }
  }
#pragma unroll
  for (int i = 0; i < kFusedPerWave; ++i) {
    const int t = i * kIdxWaves + wv;
    if (t < T) select_topk<EPL>(myl[i], lane, E, k, flags, topk_idx + (size_t)t * k, topk_w + (size_t)t * k, s_idx + t * k);
  }
  __syncthreads();
  permute_small([&](int a) { return s_idx[a]; }, T * k, n_local, offset, expert_offsets, row_src, slot_row, x, k,
                chunks_per_row, x_perm);
}

// ---- large batches: the same stable order from two short kernels over many workgroups, three from 65 workgroups on.
// (1) every workgroup ranks its own 1024 assignments (ballot inside a wavefront, serial prefix
// over its 16 wavefronts) and publishes its per-expert counts; (2) one workgroup turns the counts
// into per-(workgroup, expert) base rows (scan over workgroups, then over experts); (3) every
// workgroup adds its bases.  Up to 64 workgroups, each does (2) for itself ahead of (3) (permute_scan_place_kernel).  No atomics on the value path: the order is the unique stable one.
__global__ __launch_bounds__(kIdxThreads) void permute_rank_kernel(const int32_t* __restrict__ topk_idx, int A,
                                                                  int n_local, int offset,
                                                                  int32_t* __restrict__ block_counts,
                                                                  int32_t* __restrict__ slot_row) {
  __shared__ int32_t wave_cnt[kIdxWaves][MOE_MAX_EXPERTS];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid >> 6;
  for (int ee = lane; ee < n_local; ee += kWave) wave_cnt[wv][ee] = 0;  // (a wavefront's own row)
  const int a = blockIdx.x * kIdxThreads + tid;
  int e = -1;
  if (a < A) {
    e = topk_idx[a] - offset;
    if (e < 0 || e >= n_local) e = -1;
  }
  int count;
  const int rank = match_rank(e, lane, id_bits(n_local), count);
  if (e >= 0 && rank == 0) wave_cnt[wv][e] = count;
  __syncthreads();
  for (int ee = tid; ee < n_local; ee += kIdxThreads) {
    int run = 0;
#pragma unroll
    for (int w = 0; w < kIdxWaves; ++w) {
      const int c = wave_cnt[w][ee];
      wave_cnt[w][ee] = run;
      run += c;
    }
    block_counts[(size_t)blockIdx.x * n_local + ee] = run;
  }
  __syncthreads();
  // hand-over to the place kernel through slot_row: rank inside the workgroup (< 1024) in the low
  // 10 bits, local expert (< 256) above them
  if (a < A) slot_row[a] = (e >= 0) ? ((e << 10) | (wave_cnt[wv][e] + rank)) : -1;
}

__global__ __launch_bounds__(256) void permute_scan_kernel(int32_t* __restrict__ block_counts, int n_blocks,
                                                          int n_local, int32_t* __restrict__ expert_offsets,
                                                          int32_t* __restrict__ tickets) {
  __shared__ int32_t total[MOE_MAX_EXPERTS];
  const int tid = threadIdx.x;
  if (tickets != nullptr && tid < kTickets) tickets[tid] = 0;
  for (int e = tid; e < n_local; e += 256) {
    int run = 0;
    for (int b = 0; b < n_blocks; ++b) {
      const int c = block_counts[(size_t)b * n_local + e];
      block_counts[(size_t)b * n_local + e] = run;
      run += c;
    }
    total[e] = run;
  }
  __syncthreads();
  if (tid == 0) {
    int run = 0;
    for (int e = 0; e < n_local; ++e) {
      const int c = total[e];
      total[e] = run;
      expert_offsets[e] = run;
      run += c;
    }
    expert_offsets[n_local] = run;
  }
  __syncthreads();
  for (int i = tid; i < n_blocks * n_local; i += 256) block_counts[i] += total[i % n_local];
}

__global__ __launch_bounds__(kIdxThreads) void permute_place_kernel(int A, int n_local,
                                                                   const int32_t* __restrict__ block_bases,
                                                                   int32_t* __restrict__ row_src,
                                                                   int32_t* __restrict__ slot_row) {
  const int a = blockIdx.x * kIdxThreads + threadIdx.x;
  if (a >= A) return;
  const int v = slot_row[a];
  if (v < 0) return;
  const int e = v >> 10, rank = v & 1023;
  const int row = block_bases[(size_t)blockIdx.x * n_local + e] + rank;
  slot_row[a] = row;
  row_src[row] = a;
}

// (2) and (3) in one launch, for up to kScanBlocks workgroups: each adds up the counts of the workgroups before it and of
// all of them by itself (64 KB of counts at most, from L2; a launch saved, 4.7 us).
constexpr int kScanBlocks = 64;
__global__ __launch_bounds__(kIdxThreads) void permute_scan_place_kernel(int A, int n_local,
                                                                        const int32_t* __restrict__ block_counts,
                                                                        int32_t* __restrict__ expert_offsets,
                                                                        int32_t* __restrict__ row_src,
                                                                        int32_t* __restrict__ slot_row,
                                                                        int32_t* __restrict__ tickets) {
  __shared__ int32_t before[MOE_MAX_EXPERTS];  // rows of earlier workgroups, then this workgroup's first row
  __shared__ int32_t total[MOE_MAX_EXPERTS];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), blk = blockIdx.x, n_blocks = gridDim.x;
  const int a = blk * kIdxThreads + tid;
  const int v = a < A ? slot_row[a] : -1;
  if (blk == 0 && tickets != nullptr && tid < kTickets) tickets[tid] = 0;
  for (int e = tid; e < n_local; e += kIdxThreads) {
    int pre = 0, all = 0;
#pragma unroll 8
    for (int b = 0; b < n_blocks; ++b) {
      const int c = block_counts[(size_t)b * n_local + e];
      pre += b < blk ? c : 0;
      all += c;
    }
    before[e] = pre;
    total[e] = all;
  }
  __syncthreads();
  if (tid < kWave) {
    int carry = 0;
    for (int e0 = 0; e0 < n_local; e0 += kWave) {
      const int e = e0 + lane;
      const int c = e < n_local ? total[e] : 0;
      const int incl = gg::wave_incl_scan(c);
      if (e < n_local) {
        before[e] += carry + incl - c;
        if (blk == 0) expert_offsets[e] = carry + incl - c;
      }
      carry += __builtin_amdgcn_readlane(incl, kWave - 1);
    }
    if (blk == 0 && lane == 0) expert_offsets[n_local] = carry;
  }
  __syncthreads();
  if (v < 0) return;
  const int row = before[v >> 10] + (v & 1023);
  slot_row[a] = row;
  row_src[row] = a;
}

constexpr int kGatherThreads = 256;

__global__ __launch_bounds__(kGatherThreads) void gather_rows_kernel(const uint4* __restrict__ x,
                                                                    const int32_t* __restrict__ row_src,
                                                                    const int32_t* __restrict__ expert_offsets,
                                                                    int n_local, int k, int chunks_per_row,
                                                                    uint4* __restrict__ x_perm) {
  const int R = expert_offsets[n_local];
  for (int r = blockIdx.x; r < R; r += gridDim.x) {
    const int tok = row_src[r] / k;
    const uint4* src = x + (size_t)tok * chunks_per_row;
    uint4* dst = x_perm + (size_t)r * chunks_per_row;
    for (int c = threadIdx.x; c < chunks_per_row; c += kGatherThreads) dst[c] = src[c];
  }
}

}  // namespace

size_t permute_workspace_bytes(int T, int k, int n_local) {
  const size_t blocks = ((size_t)T * k + kIdxThreads - 1) / kIdxThreads;
  return 256 + blocks * n_local * sizeof(int32_t);
}

int32_t* permute_tickets(void* workspace, int T, int k, int n_local) {  // the last 256 bytes are nobody else's
  return reinterpret_cast<int32_t*>(static_cast<char*>(workspace) + permute_workspace_bytes(T, k, n_local) - 256);
}

size_t permute_static_counts(int T, int k, int n_local) {
  const size_t A = (size_t)T * k;
  if (A <= 2 * kIdxThreads) return 0;  // the one-workgroup path keeps its counts in LDS
  return (A + kIdxThreads - 1) / kIdxThreads * n_local;
}

hipError_t launch_permute_static(const void* x, const int32_t* topk_idx, int T, int k, int H, int n_local, int offset,
                                 void* x_perm, int32_t* expert_offsets, int32_t* row_src, int32_t* slot_row,
                                 hipStream_t stream) {
  int32_t* ptr = nullptr;
  const hipError_t err = static_scratch(&ptr);
  if (err != hipSuccess) return err;
  // every count the scan and place kernels read was written by the rank kernel of the same call:
  // nothing has to start at zero, whatever the last call left behind
  return launch_permute(x, topk_idx, T, k, H, n_local, offset, x_perm, expert_offsets, row_src, slot_row, ptr, stream);
}

static bool gathers_itself(const void* x_perm, int A, int H) { return x_perm != nullptr && (size_t)A * H * 2 <= (256u << 10); }

static hipError_t launch_gather(const void* x, const int32_t* row_src, const int32_t* expert_offsets, int A, int n_local,
                                int k, int H, void* x_perm, hipStream_t stream) {
  if (A == 0 || x_perm == nullptr) return hipSuccess;  // index only: the caller gathers on the fly
  const int grid = A < 8192 ? A : 8192;
  hipLaunchKernelGGL(gather_rows_kernel, dim3(grid), dim3(kGatherThreads), 0, stream,
                     static_cast<const uint4*>(x), row_src, expert_offsets, n_local, k, H / 8,
                     static_cast<uint4*>(x_perm));
  return hipGetLastError();
}

bool route_permute_fits(int T) {
  static_assert(kFusedTokens * MOE_MAX_TOPK <= 2 * kIdxThreads, "permute_small takes two assignments a thread");
  return T > 0 && T <= kFusedTokens;
}

hipError_t launch_route_permute(const float* logits, int T, int E, int k, uint32_t flags, int32_t* topk_idx, float* topk_w,
                                const void* x, int H, int n_local, int offset, void* x_perm, int32_t* expert_offsets,
                                int32_t* row_src, int32_t* slot_row, hipStream_t stream, int32_t* tickets) {
  const bool fuse = gathers_itself(x_perm, T * k, H);
  const auto kernel = E <= kWave ? route_permute_kernel<1> : (E <= 2 * kWave ? route_permute_kernel<2> : route_permute_kernel<4>);
  hipLaunchKernelGGL(kernel, dim3(1), dim3(kIdxThreads), 0, stream, logits, T, E, k, flags, topk_idx, topk_w, n_local, offset,
                     expert_offsets, row_src, slot_row, fuse ? static_cast<const uint4*>(x) : nullptr, H / 8,
                     static_cast<uint4*>(x_perm), tickets);
  const hipError_t err = hipGetLastError();
  if (err != hipSuccess || fuse) return err;
  return launch_gather(x, row_src, expert_offsets, T * k, n_local, k, H, x_perm, stream);
}

hipError_t launch_permute(const void* x, const int32_t* topk_idx, int T, int k, int H, int n_local, int offset,
                          void* x_perm, int32_t* expert_offsets, int32_t* row_src, int32_t* slot_row,
                          void* workspace, hipStream_t stream, int32_t* tickets) {
  const int A = T * k;
  hipError_t err;
  if (A <= 2 * kIdxThreads) {  // small batch: one workgroup does it all in one launch
    const bool fuse = gathers_itself(x_perm, A, H);
    hipLaunchKernelGGL(permute_index_kernel, dim3(1), dim3(kIdxThreads), 0, stream, topk_idx, A, n_local, offset,
                       expert_offsets, row_src, slot_row, fuse ? static_cast<const uint4*>(x) : nullptr, k, H / 8,
                       static_cast<uint4*>(x_perm), tickets);
    err = hipGetLastError();
    if (fuse) return err;
  } else {
    const int blocks = (A + kIdxThreads - 1) / kIdxThreads;
    int32_t* counts = static_cast<int32_t*>(workspace);
    hipLaunchKernelGGL(permute_rank_kernel, dim3(blocks), dim3(kIdxThreads), 0, stream, topk_idx, A, n_local, offset,
                       counts, slot_row);
    if (blocks <= kScanBlocks) {
      hipLaunchKernelGGL(permute_scan_place_kernel, dim3(blocks), dim3(kIdxThreads), 0, stream, A, n_local, counts,
                         expert_offsets, row_src, slot_row, tickets);
    } else {
      hipLaunchKernelGGL(permute_scan_kernel, dim3(1), dim3(256), 0, stream, counts, blocks, n_local, expert_offsets,
                         tickets);
      hipLaunchKernelGGL(permute_place_kernel, dim3(blocks), dim3(kIdxThreads), 0, stream, A, n_local, counts, row_src,
                         slot_row);
    }
    err = hipGetLastError();
  }
  if (err != hipSuccess) return err;
  return launch_gather(x, row_src, expert_offsets, A, n_local, k, H, x_perm, stream);
}

}  // namespace moe
