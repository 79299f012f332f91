// Block schedule for the sparse attention (Eq. 4 / Algorithm 2 take the query
// blocks in any order; this one only decides which order runs fastest).
//
// For each (b, h) the N_p blocks are sorted by a 64-bit key, ascending:
//   bits 63..33  2^30 - count      (longest list first)
//   bits 32..24  signature         (mean key position of the list, in 512ths
//                                   of N, from 8 sampled entries)
//   bits 23..0   block index       (keys are distinct: the order is unique)
// A head of more than kOrderMaxBlocks blocks is sorted in consecutive
// segments of that many blocks (each segment in place, the key holding the
// index within the segment).
// Longest-first is the classic longest-processing-time rule, so the
// workgroups of a head finish together; it also puts lists of like length
// side by side, and lists of like length walk the keys at a like pace, which
// keeps the gathers of the workgroups running together on an XCD within what
// its L2 holds.  Among lists of one length (all of them, for topK) the
// signature puts lists over like key ranges side by side.
#include <algorithm>

#include "device_common.h"
#include "launch.h"

namespace vecattn {
namespace {

// Signature of a list: its mean key position in 512ths of N, from 8 entries.
__device__ __forceinline__ int64_t sample(const int32_t* list, int64_t c, int j, int64_t N) {
  const int64_t x = list[((2 * j + 1) * c) / 16];
  return std::min<int64_t>(std::max<int64_t>(x, 0), N - 1);  // N <= 2^30: 8 of them fit
}
__device__ __forceinline__ int signature(int64_t sum, int64_t N) {
  return static_cast<int>(std::min<int64_t>((sum * 64) / N, 511));  // mean * 512 / N
}

// The signatures of all blocks, into the order array (each head's sort reads
// its own before it writes them): eight lanes per block, over the whole chip.
// The sampled entries are one cache line each, and a head's sort alone on its
// CU waited for 16384 of them at 2048 blocks: 68 us of sort then, 50 at 1182
// blocks, 16 at 512.  Heads of fewer than kSigBlocks blocks sample in the sort.
constexpr int kSigBlocks = 256;
__global__ __launch_bounds__(256) void k_signatures(const int32_t* __restrict__ idx, int64_t cap,
                                                    const int32_t* __restrict__ counts, int64_t n,
                                                    int64_t N, int32_t* __restrict__ order) {
  const int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  const int64_t r = t >> 3;
  if (r >= n) return;  // whole groups of eight lanes
  const int64_t c = std::min<int64_t>(std::max<int64_t>(counts[r], 0), cap);
  int64_t sum = c > 0 ? sample(idx + r * cap, c, static_cast<int>(t & 7), N) : 0;
#pragma unroll
  for (int o = 1; o < 8; o <<= 1) sum += __shfl_xor(static_cast<long long>(sum), o);
  if ((t & 7) == 0) order[r] = signature(sum, N);
}

// Bitonic sort of n2 = T * E keys, T threads with E consecutive ones each in
// registers: exchanges over a distance below E happen inside a thread, below
// 64 E inside a wave (lane exchanges), and only those further apart go through
// LDS and a barrier: 10 of the 66 steps at 2048 keys (all of them: 11 us more).
template <int E>
__global__ __launch_bounds__(1024) void k_attn_order(
    const int32_t* __restrict__ idx, int64_t cap, const int32_t* __restrict__ counts, int32_t Np,
    int64_t N, int32_t sampled, int32_t* order) {
  extern __shared__ uint64_t s_key[];  // [E][T]
  const int64_t bh = blockIdx.x;
  const int tid = threadIdx.x, T = blockDim.x, n2 = T * E;
  for (int64_t seg = 0; seg < Np; seg += kOrderMaxBlocks) {
    const int ns = static_cast<int>(std::min<int64_t>(Np - seg, kOrderMaxBlocks));
    const int32_t* cnt = counts + bh * Np + seg;
    int32_t* out = order + bh * Np + seg;
    uint64_t key[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
      // Keys are made by thread i % T (neighbouring lists side by side) and
      // sorted wherever they start.
      const int i = e * T + tid;
      uint64_t kk = ~uint64_t(0);  // padding sorts last
      if (i < ns) {
        const int64_t c = std::min<int64_t>(std::max<int64_t>(cnt[i], 0), cap);
        uint64_t sig = 0;
        if (sampled) {
          sig = static_cast<uint64_t>(out[i]);
        } else if (c > 0) {
          const int32_t* list = idx + (bh * Np + seg + i) * cap;
          int64_t sum = 0;
#pragma unroll
          for (int j = 0; j < 8; ++j) sum += sample(list, c, j, N);
          sig = static_cast<uint64_t>(signature(sum, N));
        }
        kk = (static_cast<uint64_t>((int64_t(1) << 30) - c) << 33) | (sig << 24) |
             static_cast<uint64_t>(i);
      }
      key[e] = kk;
    }
    // Element i = tid * E + e; ascending runs where i & k is 0.
    auto keep = [&](int e, uint64_t other, int j, int k) __attribute__((always_inline)) {
      const int i = tid * E + e;
      const bool low = ((i & j) == 0) == ((i & k) == 0);
      key[e] = low ? std::min(key[e], other) : std::max(key[e], other);
    };
    for (int k = 2; k <= n2; k <<= 1) {
      int j = k >> 1;
      for (; j >= 64 * E; j >>= 1) {
        __syncthreads();  // the exchange before has been read
#pragma unroll
        for (int e = 0; e < E; ++e) s_key[e * T + tid] = key[e];
        __syncthreads();
#pragma unroll
        for (int e = 0; e < E; ++e) keep(e, s_key[e * T + (tid ^ (j / E))], j, k);
      }
      for (; j >= E; j >>= 1) {
#pragma unroll
        for (int e = 0; e < E; ++e)
          keep(e, __shfl_xor(static_cast<unsigned long long>(key[e]), j / E), j, k);
      }
#pragma unroll
      for (int jj = E / 2; jj > 0; jj >>= 1) {
        if (jj > j) continue;
#pragma unroll
        for (int e = 0; e < E; ++e) {
          if (e & jj) continue;
          const uint64_t x = key[e], y = key[e | jj];
          const bool up = ((tid * E + e) & k) == 0;
          key[e] = up ? std::min(x, y) : std::max(x, y);
          key[e | jj] = up ? std::max(x, y) : std::min(x, y);
        }
      }
    }
    __syncthreads();  // every signature has been read
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int i = tid * E + e;
      if (i < ns) out[i] = static_cast<int32_t>(seg + static_cast<int64_t>(key[e] & 0xFFFFFF));
    }
  }
}

}  // namespace

hipError_t launch_attn_order(const int32_t* idx, int64_t cap, const int32_t* counts, int64_t rows,
                             int32_t Np, int64_t N, int32_t* order, hipStream_t stream) {
  if (rows == 0 || Np == 0) return hipSuccess;
  int n2 = 64;  // one wave at least
  while (n2 < std::min(Np, kOrderMaxBlocks)) n2 <<= 1;
  const int each = std::max(1, n2 / 1024);
  const int64_t blocks = rows * Np;
  const int sampled = Np >= kSigBlocks && (blocks + 31) / 32 <= INT32_MAX;
  if (sampled)
    hipLaunchKernelGGL(k_signatures, dim3(static_cast<unsigned>((blocks + 31) / 32)), dim3(256), 0,
                       stream, idx, cap, counts, blocks, N, order);
  auto run = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(rows)), dim3(n2 / each), n2 * 8, stream,
                       idx, cap, counts, Np, N, sampled, order);
    return hipGetLastError();
  };
  switch (each) {
    case 1: return run(k_attn_order<1>);
    case 2: return run(k_attn_order<2>);
    case 4: return run(k_attn_order<4>);
    case 8: return run(k_attn_order<8>);
    default: return run(k_attn_order<16>);
  }
}

}  // namespace vecattn
