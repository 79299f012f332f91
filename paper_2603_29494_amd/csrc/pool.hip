// Query pooling, paper Eq. 2 (Sec. 3.1.1): the pooled query of a block is the
// mean of the block's query rows.  A thread owns 8 consecutive head-dim values
// of one block and every RG-th of its rows, sums them in fp64 (bf16 values
// have 8 significant bits, so these sums are exact unless the values span more
// than ~2^38 in magnitude), adds the RG partial sums and rounds the mean to
// bf16 once.
#include <type_traits>

#include "device_common.h"
#include "launch.h"

namespace vecattn {
namespace {

// RG = 64 / (D / 8): one wave per block, a load instruction covering whole
// rows (1 KB in a row of memory) and four or eight times the waves of RG = 1
// (one thread per chunk), which small blocks keep.  Bound by the read of Q from
// 17k tokens on; below by the chain of a thread's loads.  RG = 1 / 64 rows per
// block: 1k tokens 7.2 us, 4 x 4k 10.0, 32k (28 heads) 52.8.
template <int D, int RG>
__global__ __launch_bounds__(256) void k_pool(const uint16_t* __restrict__ q, int64_t q_sB,
                                              int64_t q_sH, int64_t q_sN, int32_t H, int32_t N,
                                              int32_t P, int32_t Np, uint16_t* __restrict__ qp,
                                              int64_t p_sB, int64_t p_sH, int64_t p_sN,
                                              int64_t total) {
  constexpr int CH = D / 8;
  const int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (t >= total) return;  // whole waves with RG > 1
  const int c = static_cast<int>(t % CH);
  const int rg = static_cast<int>(t / CH % RG);
  int64_t rest = t / (CH * RG);
  const int i = static_cast<int>(rest % Np);
  rest /= Np;
  const int h = static_cast<int>(rest % H);
  const int b = static_cast<int>(rest / H);
  const int r0 = i * P;
  const int r1 = min(N, r0 + P);
  const uint16_t* base = q + b * q_sB + h * q_sH + 8 * c;
  double acc[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = 0.0;
  auto add_row = [&](const u32x4 w) __attribute__((always_inline)) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      acc[2 * e] += static_cast<double>(bf16_bits_to_f32(w[e] & 0xFFFFu));
      acc[2 * e + 1] += static_cast<double>(bf16_bits_to_f32(w[e] >> 16));
    }
  };
  // Eight rows are loaded before any is summed, so that a thread keeps eight
  // loads in flight.
  int r = r0 + rg;
  for (; r + 7 * RG < r1; r += 8 * RG) {
    u32x4 w[8];
#pragma unroll
    for (int j = 0; j < 8; ++j)
      w[j] = *reinterpret_cast<const u32x4*>(base + static_cast<int64_t>(r + j * RG) * q_sN);
#pragma unroll
    for (int j = 0; j < 8; ++j) add_row(w[j]);
  }
  // The rest, four, two and one at a time (one after another: 28 heads, 32768
  // tokens, 80-row blocks, D = 64 23.8 us against 22.9).
  auto tail = [&](auto count) __attribute__((always_inline)) {
    constexpr int n = decltype(count)::value;
    if (r + (n - 1) * RG >= r1) return;
    u32x4 w[n];
#pragma unroll
    for (int j = 0; j < n; ++j)
      w[j] = *reinterpret_cast<const u32x4*>(base + static_cast<int64_t>(r + j * RG) * q_sN);
#pragma unroll
    for (int j = 0; j < n; ++j) add_row(w[j]);
    r += n * RG;
  };
  tail(std::integral_constant<int, 4>{});
  tail(std::integral_constant<int, 2>{});
  tail(std::integral_constant<int, 1>{});
#pragma unroll
  for (int o = CH; o < CH * RG; o <<= 1)
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] += __shfl_xor(acc[e], o);
  if (rg != 0) return;
  const double n = static_cast<double>(r1 - r0);
  u32x4 out;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const uint32_t lo = f64_to_bf16_rne(acc[2 * e] / n);
    const uint32_t hi = f64_to_bf16_rne(acc[2 * e + 1] / n);
    out[e] = lo | (hi << 16);
  }
  *reinterpret_cast<u32x4*>(qp + b * p_sB + h * p_sH + static_cast<int64_t>(i) * p_sN + 8 * c) = out;
}

}  // namespace

hipError_t launch_pool(const Tensor4& q, int32_t block, void* qp, int64_t qp_sB, int64_t qp_sH,
                       int64_t qp_sN, hipStream_t stream) {
  const int32_t Np = static_cast<int32_t>((q.N + block - 1) / block);
  // Several row groups pay from a batch of eight rows each on: from 64 rows, and
  // at 32 with the four groups of D = 128.  Between those a group's rows fall
  // short of a batch: 28 heads, 32768 tokens, with groups / without, us: D = 64
  // 32 rows 31.6 / 24.1, 48 28.1 / 21.6, 64 22.5 / 31.2; D = 128 32 rows 37.0 /
  // 40.9, 48 41.2 / 38.0, 64 37.1 / 47.7.
  const bool split = block >= 64 || (block == 32 && q.D == 128);
  const int chunks = static_cast<int>(q.D / 8);
  const int64_t total = q.B * q.H * static_cast<int64_t>(Np) * (split ? 64 : chunks);
  if (total == 0) return hipSuccess;
  const int threads = 256;
  const dim3 grid(static_cast<unsigned>((total + threads - 1) / threads));
  auto run = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(threads), 0, stream, static_cast<const uint16_t*>(q.ptr),
                       q.sB, q.sH, q.sN, static_cast<int32_t>(q.H), static_cast<int32_t>(q.N),
                       block, Np, static_cast<uint16_t*>(qp), qp_sB, qp_sH, qp_sN, total);
  };
  if (q.D == 128) split ? run(k_pool<128, 4>) : run(k_pool<128, 1>);
  else split ? run(k_pool<64, 8>) : run(k_pool<64, 1>);
  return hipGetLastError();
}

}  // namespace vecattn
