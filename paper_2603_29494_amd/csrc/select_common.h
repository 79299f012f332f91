// Device-side helpers shared by the selection kernels (select.hip for long
// sequences, select_short.hip for short ones).
#pragma once

#include "device_common.h"

namespace vecattn {

// Selection modes as they come through the C ABI.
constexpr int kModeTopK = 0, kModeTopP = 1, kModeMinS = 2, kModeMinSTiled = 3;

constexpr int kMaxHeadParams = 128;  // query heads a per-head parameter list may cover
constexpr float kTopPRange = 40.0f;  // nats below the row maximum the level-0 topP bins span

__device__ __forceinline__ uint32_t ord_key(float f) {
  const uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float ord_val(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k);
}

__device__ __forceinline__ int eligible(int i, int P, int N, int causal) {
  return causal ? min(N, (i + 1) * P) : N;
}

__device__ __forceinline__ int topk_count(double r, int L) {
  int k = static_cast<int>(ceil(r * static_cast<double>(L) - 1e-9));
  return min(max(k, 1), L);
}

// exp(tau * s - ref) for topP masses (s a raw score): exp2 in fp32 while the
// exponent is in range (relative error ~1e-7), with an exact power-of-two
// rescale below it.
__device__ __forceinline__ double mass_term(float s, float tau, double ref) {
  const double y = (static_cast<double>(s) * static_cast<double>(tau) - ref) * 1.4426950408889634;
  if (y > -120.0) return static_cast<double>(__builtin_amdgcn_exp2f(static_cast<float>(y)));
  const double n = floor(y);
  return ldexp(static_cast<double>(__builtin_amdgcn_exp2f(static_cast<float>(y - n))), static_cast<int>(n));
}

// Inclusive prefix sum over the 64 lanes of a wave with DPP moves (no LDS):
// shifts by 1, 2, 4, 8 inside each 16-lane row, then row 0's total into row 1
// and row 2's into row 3 (broadcast of lane 15), and rows 0-1's total into
// rows 2-3 (broadcast of lane 31).  Lanes without a source add 0.
__device__ __forceinline__ int wave_incl_scan(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);  // row_shr:1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);  // row_shr:2
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);  // row_shr:4
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);  // row_shr:8
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // row_bcast:15
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);  // row_bcast:31
  return x;
}

// Inclusive prefix sums over the wave of a 64-bit count or an fp64 mass.
template <typename T>
__device__ __forceinline__ T wave_scan(T x) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const T y = __shfl_up(x, o);
    if (lane >= o) x += y;
  }
  return x;
}

// Orders this wave's LDS accesses on either side (a one-wave workgroup needs
// no barrier).  Unlike __syncthreads() it does not wait for the wave's
// global loads and stores: the prefetched bitmask words stay in flight and
// the stores of the lists are not waited for.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace vecattn
