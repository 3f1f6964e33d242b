// Wavefront (64 lanes) and workgroup primitives shared by the kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

typedef uint32_t u32;
typedef uint64_t u64;
typedef int64_t i64;
typedef int32_t i32;
typedef unsigned __int128 u128;
typedef __int128 i128;

#define CCLD_WAVE 64

namespace ccld {

__device__ __forceinline__ u32 lane_id() {
  return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
}

// number of set bits of m below the calling lane
__device__ __forceinline__ u32 mbcnt64(u64 m) {
  return __builtin_amdgcn_mbcnt_hi((u32)(m >> 32), __builtin_amdgcn_mbcnt_lo((u32)m, 0u));
}

// the lanes where p holds (__ballot takes an integer: the predicate would be turned into one and compared again)
__device__ __forceinline__ u64 ballot64(bool p) { return __builtin_amdgcn_ballot_w64(p); }
// the value that lane `src` (below 64) holds
__device__ __forceinline__ u32 lane_read(u32 v, u32 src) { return (u32)__builtin_amdgcn_ds_bpermute((int)(src << 2), (int)v); }
__device__ __forceinline__ i32 lane_read(i32 v, u32 src) { return __builtin_amdgcn_ds_bpermute((int)(src << 2), v); }

__device__ __forceinline__ u64 shfl_u64(u64 v, int src) {
  u32 lo = __shfl((u32)v, src, CCLD_WAVE), hi = __shfl((u32)(v >> 32), src, CCLD_WAVE);
  return ((u64)hi << 32) | lo;
}
__device__ __forceinline__ u64 shfl_xor_u64(u64 v, int m) {
  u32 lo = __shfl_xor((u32)v, m, CCLD_WAVE), hi = __shfl_xor((u32)(v >> 32), m, CCLD_WAVE);
  return ((u64)hi << 32) | lo;
}

// inclusive prefix sum over the wavefront: inside rows of 16 lanes by DPP shifts, which read zero past the row's start, then
// the sum of the row before goes to every second row and that of the lower half to the upper one.  Six instructions with
// an add each; shuffles through the LDS crossbar took six dependent trips of it.
__device__ __forceinline__ u32 wave_inclusive_sum(u32 v) {
  int x = (int)v;
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, true);       // row_shr:1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, true);       // row_shr:2
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, true);       // row_shr:4
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, true);       // row_shr:8
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false);      // row_bcast:15 into rows 1 and 3
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false);      // row_bcast:31 into rows 2 and 3
  return (u32)x;
}
__device__ __forceinline__ u32 wave_sum(u32 v) {
#pragma unroll
  for (int m = CCLD_WAVE / 2; m >= 1; m >>= 1) v += __shfl_xor(v, m, CCLD_WAVE);
  return v;
}
__device__ __forceinline__ u64 wave_max_u64(u64 v) {
#pragma unroll
  for (int m = CCLD_WAVE / 2; m >= 1; m >>= 1) { u64 o = shfl_xor_u64(v, m); v = o > v ? o : v; }
  return v;
}

// Exclusive prefix sum of one value per thread over a workgroup of THREADS threads.
// s_wave: THREADS/64 words of LDS.  *total receives the workgroup sum.  Contains barriers;
// s_wave may be reused after return.
template <int THREADS>
__device__ __forceinline__ u32 block_exclusive_sum(u32 v, u32* s_wave, u32* total) {
  constexpr int NW = THREADS / CCLD_WAVE;
  u32 lane = lane_id(), wave = threadIdx.x / CCLD_WAVE;
  u32 inc = wave_inclusive_sum(v);
  if (lane == CCLD_WAVE - 1) s_wave[wave] = inc;
  __syncthreads();
  u32 base = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) { u32 x = s_wave[w]; if ((u32)w < wave) base += x; tot += x; }
  __syncthreads();
  *total = tot;
  return base + inc - v;
}

// Waits until the wavefront's loads and stores are done.  Where a round's loads are issued conditionally one round ahead, the
// compiler cannot count what was issued behind them and waits for everything at their first use in the loop, which is
// right after the next round's loads were issued: such loops wait here, at the place that is meant.
__device__ __forceinline__ void wait_vector_memory() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// Words that workgroups of one launch hand to one another: stored and loaded past the caches that are not coherent
// between the XCDs, so that no cache has to be written back for them.
__device__ __forceinline__ void store_agent(u32* p, u32 v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void store_agent(i64* p, i64 v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ i64 load_agent(const i64* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ u32 load_agent(const u32* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
// True in the last of `blocks` workgroups to get here.  What the others stored with store_agent or added with atomics
// before is there for load_agent: the barrier waits until a wavefront's stores are done.  (A release fence in every thread
// would write the L2 back once per wavefront: 40 us over the 4,096 wavefronts of a counting pass.)  s_last: a word of LDS.
__device__ __forceinline__ bool last_block(u32* done, u32 blocks, u32* s_last) {
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (threadIdx.x == 0) *s_last = atomicAdd(done, 1u) + 1 == blocks;
  __syncthreads();
  return *s_last != 0;
}

// The same with the arrivals counted in two levels, each counter in a line of its own: atomics on one word follow one another at
// 35 to 50 ns each, so 1,200 workgroups would take 50 us to arrive.  words: ARRIVAL_WORDS of them, zero before and behind.
constexpr u32 ARRIVAL_GROUPS = 16, ARRIVAL_STRIDE = 32, ARRIVAL_WORDS = (ARRIVAL_GROUPS + 1) * ARRIVAL_STRIDE;
__device__ __forceinline__ bool last_arrival(u32* words, u32 blocks, u32* s_last) {
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (threadIdx.x == 0) {
    const u32 g = blockIdx.x % ARRIVAL_GROUPS, members = (blocks - g + ARRIVAL_GROUPS - 1) / ARRIVAL_GROUPS;
    const u32 groups = blocks < ARRIVAL_GROUPS ? blocks : ARRIVAL_GROUPS;
    u32* const mine = words + (g + 1) * ARRIVAL_STRIDE;
    bool last = atomicAdd(mine, 1u) + 1 == members;
    if (last) {
      store_agent(mine, 0u);
      last = atomicAdd(words, 1u) + 1 == groups;
      if (last) store_agent(words, 0u);
    }
    *s_last = last;
  }
  __syncthreads();
  return *s_last != 0;
}

}  // namespace ccld
