// device_common.h - small device helpers shared by the gfx950 kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace chimera {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;

// 2^22: one unit of an inner product of two grid vectors is 2^-22.
#define KEY_SCALE 4194304.0f

__device__ __forceinline__ bf16x8 as_bf16x8(uint4 v) { return __builtin_bit_cast(bf16x8, v); }

// Value grid: nearest multiple of max(2^-11, bf16 spacing), ties to even.
__device__ __forceinline__ uint16_t grid_bf16_bits(float x) {
  if (fabsf(x) < 0.0625f) {
    float g = rintf(x * 2048.0f) * (1.0f / 2048.0f);  // exact: |g| <= 2^-4, <= 8 significant bits
    return (uint16_t)(__float_as_uint(g) >> 16);
  }
  uint32_t u = __float_as_uint(x);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// Order-preserving 64-bit key of (score desc, id asc): larger is better.
__device__ __forceinline__ uint64_t pack_key(int32_t score_key, uint32_t id) {
  return ((uint64_t)((uint32_t)score_key ^ 0x80000000u) << 32) | (uint64_t)(0xFFFFFFFFu - id);
}
__device__ __forceinline__ int32_t key_score(uint64_t k) { return (int32_t)((uint32_t)(k >> 32) ^ 0x80000000u); }
__device__ __forceinline__ uint32_t key_id(uint64_t k) { return 0xFFFFFFFFu - (uint32_t)k; }

// Exact conversion of a grid inner product (fp32, a multiple of 2^-22 below
// 2^2 in magnitude) to its integer key.
__device__ __forceinline__ int32_t to_key(float s) { return (int32_t)(s * KEY_SCALE); }

__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & 63); }

// F' of a document outside the candidate set S_Q (a real F' is never this small).
constexpr int NO_HIT = (int)0x80000000;
// Bins of the first radix pass of the refinement select (top 12 key bits).
constexpr int SEL_BINS = 4096;

// Unsigned order key of a partial score: larger F' <-> larger key.
__device__ __forceinline__ uint32_t fp_key(int32_t f) { return (uint32_t)f ^ 0x80000000u; }

// First position p in [lo, hi) of the ascending array a with a[p] >= x.
__device__ __forceinline__ int64_t lower_bound_i32(const int32_t *__restrict__ a, int64_t lo, int64_t hi, int64_t x) {
  while (lo < hi) {
    const int64_t mid = lo + ((hi - lo) >> 1);
    if ((int64_t)a[mid] < x) lo = mid + 1; else hi = mid;
  }
  return lo;
}

// Inclusive prefix sum over the 64 lanes of a wave, by DPP adds.
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t x) {
  int v = (int)x;
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);  // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);  // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);  // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);  // row_shr:8
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);  // row_bcast:15 into rows 1, 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);  // row_bcast:31 into rows 2, 3
  return (uint32_t)v;
}

// Maximum over the 64 lanes of a wave, in every lane, by DPP moves.
__device__ __forceinline__ uint64_t wave_max_u64(uint64_t x) {
#define CHIMERA_MX64(CTRL, ROWS)                                                                              \
  {                                                                                                           \
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)x, CTRL, ROWS, 0xF, false);   \
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(x >> 32), CTRL, ROWS, 0xF, false);     \
    const uint64_t y = (uint64_t)hi << 32 | lo;                                                               \
    x = y > x ? y : x;                                                                                        \
  }
  CHIMERA_MX64(0x111, 0xF)  // row_shr:1, 2, 4, 8: lane 15 of each row of 16
  CHIMERA_MX64(0x112, 0xF)
  CHIMERA_MX64(0x114, 0xF)
  CHIMERA_MX64(0x118, 0xF)
  CHIMERA_MX64(0x142, 0xA)  // row_bcast:15 into rows 1, 3
  CHIMERA_MX64(0x143, 0xC)  // row_bcast:31 into rows 2, 3
#undef CHIMERA_MX64
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, 63);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(x >> 32), 63);
  return (uint64_t)hi << 32 | lo;
}

// Exclusive prefix sum of x over a block of W waves and the total.  wsum [W]
// is shared and free for the next call once every thread has passed a barrier
// after this one.
template <int W>
__device__ __forceinline__ uint32_t block_scan(uint32_t x, uint32_t *wsum, uint32_t &total) {
  const uint32_t incl = wave_incl_scan(x);
  if (lane_id() == 63) wsum[threadIdx.x >> 6] = incl;
  __syncthreads();
  uint32_t base = 0, all = 0;
#pragma unroll
  for (int w = 0; w < W; ++w) {
    const uint32_t y = wsum[w];
    base += w < (int)(threadIdx.x >> 6) ? y : 0;
    all += y;
  }
  total = all;
  return base + incl - x;
}

// Radix-select step over the 64 W PER bins of `bins` (16-byte aligned), from the
// highest bin down, by a block of W waves: the bin where the running count
// reaches rem (0 < rem <= total), the count above it and its own; without such
// a bin (total < rem) found stays as it was.  Returns the total.  found and wsum
// are shared; both are free for the next call after a barrier.
template <int W, int PER>
__device__ __forceinline__ uint32_t find_bin(const uint32_t *bins, uint32_t rem, uint32_t *wsum, uint3 *found) {
  static_assert(PER % 4 == 0, "whole 16-byte groups");
  const int top = 64 * W * PER - PER * ((int)threadIdx.x + 1);  // this thread's bins: top + PER - 1 down to top
  uint32_t x[PER], sum = 0;
#pragma unroll
  for (int i = 0; i < PER; i += 4) {
    const uint4 y = *(const uint4 *)(bins + top + i);
    x[i] = y.x;
    x[i + 1] = y.y;
    x[i + 2] = y.z;
    x[i + 3] = y.w;
    sum += y.x + y.y + y.z + y.w;
  }
  uint32_t total;
  uint32_t cum = block_scan<W>(sum, wsum, total);
  if (cum < rem && cum + sum >= rem) {
#pragma unroll
    for (int i = PER - 1; i >= 0; --i) {
      if (cum < rem && cum + x[i] >= rem) *found = make_uint3((uint32_t)(top + i), cum, x[i]);
      cum += x[i];
    }
  }
  __syncthreads();
  return total;
}

template <class T>
__device__ __forceinline__ T shfl_xor(T v, int m) {
  return __shfl_xor(v, m, 64);
}

__device__ __forceinline__ uint64_t shfl_xor_u64(uint64_t v, int m) {
  uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
  lo = __shfl_xor(lo, m, 64);
  hi = __shfl_xor(hi, m, 64);
  return ((uint64_t)hi << 32) | lo;
}

}  // namespace chimera
