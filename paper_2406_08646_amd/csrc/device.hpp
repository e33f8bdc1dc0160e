// Device-side building blocks: wave/block reductions, XCD-aware block
// order and the deterministic "last workgroup finishes the reduction"
// pattern used by the fused solver kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace spx {

// v from the lane R places on in each row of 16 lanes (rotating).
template <int R>
__device__ __forceinline__ double row_rotate(double v) {
  return __builtin_amdgcn_update_dpp(0.0, v, 0x120 + R, 0xf, 0xf, true);
}

// v + v of the lane 32 (HALF) or 16 places away.
template <bool HALF>
__device__ __forceinline__ double swap_add(double v) {
  const uint64_t b = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)b, hi = (uint32_t)(b >> 32);
  // each swap leaves the lower half's (even row's) word in one result and
  // the upper half's (odd row's) in the other, in both places
  auto l = HALF ? __builtin_amdgcn_permlane32_swap(lo, lo, false, false)
                : __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
  auto h = HALF ? __builtin_amdgcn_permlane32_swap(hi, hi, false, false)
                : __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
  return __longlong_as_double((long long)(((uint64_t)h[0] << 32) | l[0])) +
         __longlong_as_double((long long)(((uint64_t)h[1] << 32) | l[1]));
}

// Sum over the 64 lanes of a wave; every lane receives the total.  The
// order is fixed (lane l adds lane l ^ 32's value, then l ^ 16's, ... l ^
// 1's), so the result is reproducible.  The steps stay in the vector unit:
// half and row swaps, then rotations in a row of 16, which reach lane l ^ d
// for d = 8, 4, 2, 1 because by then the sums repeat every 2 d lanes.  The
// same butterfly through LDS permutes (__shfl_xor) is on the critical path
// of every dot: a resident CG iteration on 66,049 rows took 6.8 us with it
// and takes 6.35 now, on 4,225 rows 5.0 and 4.4; 512 small systems in one
// batch 7.24 and 6.96 ms; an fp32 inner iteration on 884,736 rows 1.6% less.
__device__ __forceinline__ double wave_sum(double v) {
  v = swap_add<true>(v);
  v = swap_add<false>(v);
  v += row_rotate<8>(v);
  v += row_rotate<4>(v);
  v += row_rotate<2>(v);
  v += row_rotate<1>(v);
  return v;
}

// Sum over aligned groups of L lanes (L a power of two <= 64); every lane of
// the group receives the group total.
template <int L, typename T>
__device__ __forceinline__ T group_sum(T v) {
#pragma unroll
  for (int off = L / 2; off >= 1; off >>= 1) v += __shfl_xor(v, off, L);
  return v;
}

// Block-wide sum for blockDim.x == BLOCK; the result is valid in thread 0.
template <int BLOCK>
__device__ __forceinline__ double block_sum(double v, double* lds) {
  static_assert(BLOCK % 64 == 0, "block must be whole waves");
  v = wave_sum(v);
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (lane == 0) lds[w] = v;
  __syncthreads();
  double r = 0.0;
  if (threadIdx.x == 0) {
#pragma unroll
    for (int i = 0; i < BLOCK / 64; ++i) r += lds[i];
  }
  __syncthreads();
  return r;
}

// Workgroups are dispatched round-robin over the 8 XCDs (block b lands on
// XCD b % 8).  Renumber them so every XCD walks one contiguous range of
// logical blocks, which keeps neighbouring rows (and the x entries they
// share) in one L2.  Bijective for any block count.
__device__ __forceinline__ int64_t xcd_logical_block(int64_t b, int64_t nb) {
  const int64_t q = nb >> 3, r = nb & 7;
  const int64_t x = b & 7, i = b >> 3;
  return x * q + (x < r ? x : r) + i;
}

// Loads that bypass the L2 allocation policy for streamed matrix data.
template <typename T>
__device__ __forceinline__ T stream_load(const T* p) {
  return __builtin_nontemporal_load(p);
}

}  // namespace spx
