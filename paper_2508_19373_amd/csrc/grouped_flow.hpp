// Streaming tiles: grouped "NT" GEMM for experts of up to about 160 rows, in places two passes of them (flow_plan in
// expert_ffn.hip says where it runs) (gfx950), bound: HBM.
//
// Up to there a grouped GEMM is bound by streaming every active expert's weights once.  One
// workgroup per tile (grouped_gemm.hpp) spends a fifth to a third of such a tile's time outside its k-loop: finding the
// tile, filling the LDS stages, the epilogue and the gap to the next workgroup, during all of which its compute
// unit has little or nothing in flight.  Here a workgroup stays and takes tile after tile, and the weight stream never stops:
//  * eight wavefronts, four that multiply and four that only issue the LDS-DMA loads.  The loaders run NSB - 1 k-tiles
//    ahead of the multipliers, across tile boundaries: the next tile's first k-tiles are in flight while this one's
//    last are multiplied and stored.  A wavefront's wait counts see its own loads only, so the multipliers' stores
//    and look-ups never wait for the stream, nor the stream for them;
//  * one barrier per k-tile for all eight: before it the loaders have waited for the k-tile it opens, the multipliers are
//    done with the one before, whose stages the loaders refill behind it;
//  * the multipliers' first wavefront looks up tiles ahead of time and leaves them (coordinates, source rows) in a
//    ring of slots in LDS, from the prefix of tiles per expert computed once per workgroup;
//  * an expert's row passes are of one height and multiply the 32-row pairs of blocks that hold rows, no more (skewed
//    batches: Mixtral EP=2 under Zipf(1.2), 450 tokens, layer 429 -> 419 us, the cold shard of Qwen2-57B TP=2 EP=2 at 1000 404 ->
//    392; equal where all passes are full);
//  * tiles are taken from a counter where the caller has one (cleared by an earlier kernel of the same stream), so that a
//    workgroup that starts late, behind another stream's kernel, takes fewer; else dealt round-robin.
// Nothing waits for another workgroup.
#pragma once
#include <type_traits>

#include "flow_tiles.hpp"
#include "moe_internal.hpp"
#include "unit_list_wave.hpp"

namespace moe {
namespace gf {

constexpr int BK = 64;           // K elements per LDS row (128 bytes, 8 chunks of 16 bytes)
constexpr int kMul = 4, kLoad = 4;  // wavefronts that multiply / that load
constexpr int kThreads = (kMul + kLoad) * 64;
constexpr int kSlots = 4;        // ring of looked-up tiles

typedef __attribute__((address_space(3))) void lds_void_t;
typedef __attribute__((address_space(1))) const void global_void_t;

__device__ __forceinline__ int swz(int row) { return (row >> 1) & 7; }
__device__ __forceinline__ int lds_off(int row, int chunk) { return row * BK + ((chunk ^ swz(row)) << 3); }
__device__ __forceinline__ float silu_mul(float g, float u) { return g * __builtin_amdgcn_rcpf(1.f + __expf(-g)) * u; }

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}
// The barrier of a k-tile: the wavefront's LDS accesses are done before it, and none is moved across it.
__device__ __forceinline__ void barrier() {
#ifdef __HIP_DEVICE_COMPILE__
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#endif
}

// LDS stages: as many weight stages as fit beside the activation stages and the tile slots.
template <int BM, int BN>
struct Shape {
  static constexpr int kStageA = BM * BK, kStageB = BN * BK;  // elements
  static constexpr int NSA = BN >= 256 ? 3 : 6;
  static constexpr int NSB = BN >= 256 ? (BM >= 128 ? 3 : 4) : NSA;
  static_assert(NSA <= NSB, "the weights run ahead at least as far as the activations");
  static_assert((NSA * kStageA + NSB * kStageB) * 2 <= (160 - 4) * 1024, "LDS budget, beside the tile slots");
  static constexpr int kRowsA = BM / 8, kRowsB = BN / 8;      // 1 KB DMA instructions per k-tile
  static constexpr int A_INST = (kRowsA + kLoad - 1) / kLoad, B_INST = kRowsB / kLoad;
  static_assert(kRowsB % kLoad == 0 && (kRowsA % kLoad == 0), "whole instructions per loader");
  // loads that may be in flight at the barrier that opens a k-tile: those issued after the last that it needs, its
  // activations or (with as many stages of each) its weights
  static constexpr int kSlack = (NSA < NSB ? B_INST : 0) + (NSA - 2) * (A_INST + B_INST);
  static_assert(kSlack < 64, "the wait count has six bits");
};

struct Slot {
  int expert, row0, row_end;  // expert < 0: no more tiles; row_end - row0 <= BM
  int strip0, strips;         // its 16-column output strips
  int kt0;                    // the k-tile its walk over K begins with
};

// Weight rows are addressed as a buffer from the tile's first row on; loads at kBufBytes and above bring nothing and
// cost no memory access, which is how a tile narrower than BN leaves out the rest (its wait counts stay the same).
constexpr uint32_t kBufBytes = 0x80000000u;
#ifdef __HIP_DEVICE_COMPILE__
typedef __amdgpu_buffer_rsrc_t buf_t;
__device__ __forceinline__ buf_t make_buf(const void* p) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, kBufBytes, 0x00027000);
}
__device__ __forceinline__ void buf_to_lds(buf_t b, lds_void_t* dst, uint32_t lane_off, uint32_t off) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(b, dst, 16, lane_off, off, 0, 0);
}
#else
struct buf_t {};
__device__ inline buf_t make_buf(const void*) { return buf_t{}; }
__device__ inline void buf_to_lds(buf_t, lds_void_t*, uint32_t, uint32_t) {}
#endif

// Measured (weights in no cache): Qwen1.5-MoE, 60 experts of 22 rows, gate/up 692 MB 140 -> 125 us (5.5 TB/s), down 86 ->
// 68 (5.1); TP=4 slice of Mixtral, 14 rows, 96 -> 83 (5.7) and 52 -> 45; against one workgroup per 64-row tile and the
// streaming kernel.  About 5 us of a launch are not the stream: start, first look-up, first and last tile.
// grid = any number of workgroups (one per compute unit); GATEUP: B0 = gate, B1 = up, C = h (bf16); else B0 = down.
// regions, step: k_regions and k_step, of which the tiles' walks over K take their begin.  Requires K % 64 == 0, 192 <= K <= 2^21 and n_out % 16 == 0.
template <int BM, int BN, bool GATEUP, typename OutT>
__global__ __launch_bounds__(kThreads, 2) void grouped_flow_kernel(
    const uint16_t* __restrict__ A, const int32_t* __restrict__ expert_offsets, int n_local,
    int regions, uint32_t step, const uint16_t* __restrict__ B0, const uint16_t* __restrict__ B1, int n_out, int K, OutT* __restrict__ C,
    const RowMap rows, int32_t* __restrict__ ticket) {
  using S = Shape<BM, BN>;
  constexpr int NSA = S::NSA, NSB = S::NSB;
  constexpr int TM = BM / 16, TN = BN / kMul / 16;
  static_assert(!GATEUP || TN % 2 == 0, "gate and up blocks pair up inside a wavefront");
  __shared__ __attribute__((aligned(1024))) uint16_t stages[NSA * S::kStageA + NSB * S::kStageB];
  __shared__ int s_pre[MOE_MAX_EXPERTS];        // row passes before each expert
  __shared__ Slot s_slot[kSlots];
  __shared__ int s_row[kSlots][BM];             // source row of each of a tile's rows

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nk = K / BK;
  const int strips = n_out / 16;
  int ncb = 1;  // tiles a (expert, row pass) is cut into
  const int pace = look_pace(nk), ahead = look_ahead(nk, NSB);
  static_assert(look_ahead(3, NSB) < kSlots && look_ahead(16, NSB) < kSlots, "the tile in work keeps its slot");

  // ---- once: the prefix of tiles per expert
  const int chunks = (n_local + 63) >> 6;
  int total = 0;
  int taken = 0;  // tiles this workgroup has taken
  auto take = [&]() {
    const int n = taken++;
    if (ticket == nullptr) return (int)blockIdx.x + n * (int)gridDim.x;
    int t = 0;
    if (lane == 0) t = atomicAdd(ticket, 1);
    return t;  // of lane 0
  };
  int pending = 0;
  auto find = [&](int id, Slot& s) {
    s.expert = -1;
    s.row0 = s.row_end = s.strip0 = s.strips = s.kt0 = 0;
    // The row passes of a column tile are neighbours in the list, and so on one XCD: they walk K together and the later
    // readers of its weights find them in that XCD's L2.
    id = tile_place(id, total);
    if (id < 0) return;
    int before = 0;
#pragma unroll
    for (int j = 0; j < gg::kLaneChunks; ++j) {
      if (j < chunks) {
        const int e = j * 64 + lane;
        before += __popcll(__ballot(e < n_local && s_pre[min(e, n_local - 1)] * ncb <= id));
      }
    }
    const int e = before - 1;  // the last expert that starts at or before it
    const int lo = expert_offsets[e], hi = expert_offsets[e + 1];
    const int local = id - __builtin_amdgcn_readfirstlane(s_pre[e]) * ncb;
    // the row passes of an expert are of one height, and multiply no more than that: an expert of 215 rows is two passes of 112
    const int passes = (hi - lo + BM - 1) / BM, height = ((hi - lo + passes - 1) / passes + 15) & ~15;
    const int nb = local / passes;
    s.expert = e;
    s.strip0 = nb * strips / ncb;
    s.strips = (nb + 1) * strips / ncb - s.strip0;
    s.row0 = lo + (local - nb * passes) * height;
    // The walks over K begin apart: workgroups that all stand at the same k read the same 128 bytes of rows 4 or 8 KB
    // apart, which fall on a few of the memory channels (gate/up of Qwen1.5-MoE, K = 2048, 22 rows per expert 138 us from k = 0,
    // 126 so; TP=4 slice of Mixtral, K = 4096, 94 and 84; K = 1408 and 3584 no difference.  Begins by the tile's place in the
    // list, which the other rows decide, were no faster: 126 and 85).  With 128 rows and more, where an XCD's tiles share as
    // much of the activations as of the weights, eight places and not 16 (90 rows: 139 us, 152 from 16).
    s.kt0 = k_first(e, nb, ncb, regions, step);
    s.row_end = min(hi, s.row0 + height);
  };
  // source rows of a tile's rows, the last valid one behind its end
  auto source_row = [&](const Slot& s, int r) { return rows(min(s.row0 + r, s.row_end - 1)); };
  auto publish = [&](int slot, const Slot& s, const int (&src)[(BM + 63) / 64]) {
    if (lane == 0) s_slot[slot] = s;
#pragma unroll
    for (int q = 0; q < (BM + 63) / 64; ++q)
      if (q * 64 + lane < BM) s_row[slot][q * 64 + lane] = src[q];
  };
  if (wave == 0) {
    int first = take();  // (in flight together with the offsets)
    int len[gg::kLaneChunks], pre[gg::kLaneChunks];
#pragma unroll
    for (int j = 0; j < gg::kLaneChunks; ++j) {
      const int e = j * 64 + lane;
      const bool ok = j < chunks && e < n_local;
      const int lo = ok ? expert_offsets[e] : 0, hi = ok ? expert_offsets[e + 1] : 0;
      len[j] = (hi - lo + BM - 1) / BM;
    }
    const int units = gg::wave_prefix(len, chunks, pre);
    // tiles of equal width, as many as leave none of this launch's workgroups idle in the last round: lane l prices
    // fewest + l * regions.  Dealt in turn to 240 workgroups, the price for 256 left a fifth of the launch idle (gate/up of 15
    // experts of Qwen1.5-MoE, 30 rows each, 49 / 35 us, 60 of 22 134 / 129, TP=4 slice of Mixtral 111 / 84).  From the counter the
    // workgroups that run beside the other stream's are neither all of the launch nor the same ones throughout, and narrow
    // tiles even that out: priced as a full launch (layer of Qwen2-57B, 450 tokens, 898, at the price for 240 950; Qwen1.5-MoE 333:
    // 259 and 265).
    const int wgs = ticket == nullptr ? (int)gridDim.x : workgroups(false);
    {
      const int fewest = fewest_tiles(strips, BN, GATEUP, regions), n = fewest + lane * regions;
      const float cost = n <= strips ? tile_cost_of(units, wgs, strips, n, BM, BN, GATEUP) : 3e38f;
      float best = cost;
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) best = fminf(best, __shfl_xor(best, o, 64));
      ncb = __builtin_amdgcn_readfirstlane(fewest + (__ffsll((long long)__ballot(cost == best)) - 1) * regions);
    }
    total = units * ncb;
#pragma unroll
    for (int j = 0; j < gg::kLaneChunks; ++j)
      if (j < chunks && j * 64 + lane < n_local) s_pre[j * 64 + lane] = pre[j];
    for (int n = 0; n < ahead; ++n) {
      const int id = __builtin_amdgcn_readfirstlane(n == 0 ? first : take());
      Slot s;
      find(id, s);
      int src[(BM + 63) / 64];
#pragma unroll
      for (int q = 0; q < (BM + 63) / 64; ++q) src[q] = s.expert >= 0 ? source_row(s, q * 64 + lane) : 0;
      publish(n, s, src);
    }
  }
  barrier();

  if (wave >= kMul) {
    // ---- loaders: DMA instruction j of loader w brings 8 rows of 128 bytes, row (j * kLoad + w) * 8 + lane / 8 of the
    // tile, chunk lane % 8 as the swizzle places it
    const int w = wave - kMul;
    const int dma_row = lane >> 3, dma_chunk = (lane & 7) ^ swz(w * 8 + dma_row);
    static_assert(kLoad % 2 == 0, "a loader's instructions start at rows with the same swizzle");
    const uint16_t* a_src[S::A_INST];
    buf_t b_buf;
    uint32_t b_lane[S::B_INST];  // lane offsets of the weight rows; kBufBytes where the tile ends before them
    const uint32_t b_row = (uint32_t)dma_row * (uint32_t)K * 2u + (uint32_t)dma_chunk * 16u;
    int ta = 0, ka = 0, tb = 0, kb = 0;   // next k-tile to load: tile (of this workgroup) and how many k-tiles of it are
    int ca = 0, cb = 0;                   // loaded; its place in K
    bool more_a, more_b;
    auto open_a = [&](int t) {
      const int sl = t & (kSlots - 1);
      more_a = __builtin_amdgcn_readfirstlane(s_slot[sl].expert) >= 0;
      ca = __builtin_amdgcn_readfirstlane(s_slot[sl].kt0);
      const int live = (__builtin_amdgcn_readfirstlane(s_slot[sl].row_end - s_slot[sl].row0) + 31) & ~31;
#pragma unroll
      for (int j = 0; j < S::A_INST; ++j) {
        // rows that are not multiplied: one 16-byte piece for the whole instruction
        const int r = (j * kLoad + w) * 8 + dma_row, chunk = (j * kLoad + w) * 8 < live ? dma_chunk : 0;
        a_src[j] = A + (size_t)s_row[sl][r] * K + chunk * 8;
      }
    };
    auto open_b = [&](int t) {
      const int sl = t & (kSlots - 1);
      const int e = __builtin_amdgcn_readfirstlane(s_slot[sl].expert);
      const int strip0 = __builtin_amdgcn_readfirstlane(s_slot[sl].strip0);
      const int n = __builtin_amdgcn_readfirstlane(s_slot[sl].strips);
      more_b = e >= 0;
      cb = __builtin_amdgcn_readfirstlane(s_slot[sl].kt0);
      // 16-row blocks alternate gate, up, gate, up ... of the same output columns: a loader's instructions are 32 rows
      // apart, all in one matrix
      static_assert(kLoad * 8 == 32, "one matrix per loader");
      const uint16_t* m = GATEUP && (w & 2) ? B1 : B0;
      b_buf = make_buf(m + ((size_t)max(e, 0) * n_out + (size_t)strip0 * 16) * K);
#pragma unroll
      for (int j = 0; j < S::B_INST; ++j) {
        const int r = GATEUP ? j * 16 + (w & 1) * 8 : (j * kLoad + w) * 8;
        b_lane[j] = r < n * 16 ? b_row + (uint32_t)r * (uint32_t)K * 2u : kBufBytes;
      }
    };
    int sa = 0, sb = 0;  // stages they go to
    auto load_a = [&]() {
      if (!more_a) return;
#pragma unroll
      for (int j = 0; j < S::A_INST; ++j)
        __builtin_amdgcn_global_load_lds((global_void_t*)(a_src[j] + (size_t)ca * BK),
                                         (lds_void_t*)(stages + sa * S::kStageA + (j * kLoad + w) * 8 * BK), 16, 0, 0);
      sa = sa + 1 == NSA ? 0 : sa + 1;
      ca = ca + 1 == nk ? 0 : ca + 1;
      if (++ka == nk) {
        ka = 0;
        open_a(++ta);
      }
    };
    auto load_b = [&]() {
      if (!more_b) return;
#pragma unroll
      for (int j = 0; j < S::B_INST; ++j)
        buf_to_lds(b_buf, (lds_void_t*)(stages + NSA * S::kStageA + sb * S::kStageB + (j * kLoad + w) * 8 * BK),
                   b_lane[j], cb * (BK * 2));
      sb = sb + 1 == NSB ? 0 : sb + 1;
      cb = cb + 1 == nk ? 0 : cb + 1;
      if (++kb == nk) {
        kb = 0;
        open_b(++tb);
      }
    };
    open_a(0);
    open_b(0);
    // what the k-tiles before the first would have issued, in their order
    for (int g = 1 - NSB; g < 0; ++g) {
      if (g + NSA > 0) load_a();
      load_b();
    }
    // (at k-tile g: the activations of k-tile g - 1 + NSA and the weights of g - 1 + NSB, behind the barrier that opens g;
    // at the end, with nothing left to issue, the wait is for everything)
    for (int t = 0; __builtin_amdgcn_readfirstlane(s_slot[t & (kSlots - 1)].expert) >= 0; ++t) {
      for (int kt = 0; kt < nk; ++kt) {
        if (more_b)
          wait_vmcnt<S::kSlack>();
        else
          wait_vmcnt<0>();
        barrier();
        load_a();
        load_b();
      }
    }
    return;
  }

  // ---- multipliers: wavefront w has weight rows [w * BN / 4, ...) of the tile and all of its BM rows
  const int lrow = lane & 15, kq = lane >> 4;
  int sa = 0, sb = 0;
  Slot nxt;
  nxt.expert = -1;
  int nsrc[(BM + 63) / 64] = {};
  for (int t = 0;; ++t) {
    Slot cur;
    cur.expert = __builtin_amdgcn_readfirstlane(s_slot[t & (kSlots - 1)].expert);
    if (cur.expert < 0) break;
    cur.row0 = __builtin_amdgcn_readfirstlane(s_slot[t & (kSlots - 1)].row0);
    cur.row_end = __builtin_amdgcn_readfirstlane(s_slot[t & (kSlots - 1)].row_end);
    cur.strip0 = __builtin_amdgcn_readfirstlane(s_slot[t & (kSlots - 1)].strip0);
    cur.strips = __builtin_amdgcn_readfirstlane(s_slot[t & (kSlots - 1)].strips);
    const int pairs = (cur.row_end - cur.row0 + 31) >> 5;  // of 16-row blocks that hold rows
    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int kt = 0; kt < nk; ++kt) {
      barrier();
      const uint16_t* pa = stages + sa * S::kStageA;
      const uint16_t* pb = stages + NSA * S::kStageA + sb * S::kStageB;
      bf16x8 bfr[TN][2];
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          bfr[j][ks] = *reinterpret_cast<const bf16x8*>(pb + lds_off(wave * (BN / kMul) + j * 16 + lrow, ks * 4 + kq));
      // Pairs of 16-row blocks, as many as hold rows; a pair's operands are read in front of the MFMAs of the one before.
      // (A version of the whole k-tile per height spills: the accumulators change registers between them.)
      static_assert(TM % 2 == 0, "row blocks in pairs");
      bf16x8 af[2][2][2];
      auto read_pair = [&](auto p_tag) {
        constexpr int p = decltype(p_tag)::value;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int ks = 0; ks < 2; ++ks)
            af[p & 1][h][ks] = *reinterpret_cast<const bf16x8*>(pa + lds_off((p * 2 + h) * 16 + lrow, ks * 4 + kq));
      };
      auto pair_from = [&](auto self, auto p_tag) {
        constexpr int p = decltype(p_tag)::value;
        if constexpr (p < TM / 2) {
          if (p == 0 || p < pairs) {
            if constexpr (p + 1 < TM / 2) read_pair(std::integral_constant<int, p + 1>{});
#pragma unroll
            for (int h = 0; h < 2; ++h)
              // weights as the MFMA "A" operand: a lane ends up with 4 consecutive output columns of one row
#pragma unroll
              for (int j = 0; j < TN; ++j) {
                f32x4& c = acc[p * 2 + h][j];
                c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[j][0], af[p & 1][h][0], c, 0, 0, 0);
                c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[j][1], af[p & 1][h][1], c, 0, 0, 0);
              }
            self(self, std::integral_constant<int, p + 1>{});
          }
        }
      };
      read_pair(std::integral_constant<int, 0>{});
      pair_from(pair_from, std::integral_constant<int, 0>{});
      sa = sa + 1 == NSA ? 0 : sa + 1;
      sb = sb + 1 == NSB ? 0 : sb + 1;
      if (wave == 0) {  // the look-up of tile t + ahead
        if (kt == 0) pending = take();
        if (kt == pace) {
          find(__builtin_amdgcn_readfirstlane(pending), nxt);
#pragma unroll
          for (int q = 0; q < (BM + 63) / 64; ++q) nsrc[q] = nxt.expert >= 0 ? source_row(nxt, q * 64 + lane) : 0;
        }
        if (kt == 2 * pace) publish((t + ahead) & (kSlots - 1), nxt, nsrc);
      }
    }
    // ---- epilogue: accumulator register v of block (i, j) is row i * 16 + lane % 16, column j * 16 + (lane / 16) * 4 + v
    constexpr int JS = GATEUP ? 2 : 1;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int row = cur.row0 + i * 16 + lrow;
#pragma unroll
      for (int j = 0; j < TN; j += JS) {
        const int strip = GATEUP ? (wave * TN + j) / 2 : wave * TN + j;
        const int col = (cur.strip0 + strip) * 16 + kq * 4;
        if (row < cur.row_end && strip < cur.strips) {
          const f32x4& v = acc[i][j];
          if constexpr (GATEUP) {
            const f32x4& u = acc[i][j + 1];
            uint2 o;
            o.x = pack_bf16x2(silu_mul(v[0], u[0]), silu_mul(v[1], u[1]));
            o.y = pack_bf16x2(silu_mul(v[2], u[2]), silu_mul(v[3], u[3]));
            *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(C) + (size_t)row * n_out + col) = o;
          } else if constexpr (sizeof(OutT) == 4) {
            *reinterpret_cast<float4*>(C + (size_t)row * n_out + col) = make_float4(v[0], v[1], v[2], v[3]);
          } else {
            uint2 o;
            o.x = pack_bf16x2(v[0], v[1]);
            o.y = pack_bf16x2(v[2], v[3]);
            *reinterpret_cast<uint2*>(C + (size_t)row * n_out + col) = o;
          }
        }
      }
    }
  }
}

}  // namespace gf
}  // namespace moe
