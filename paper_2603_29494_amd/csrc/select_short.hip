// Important-vector selection for short sequences (N <= kShortMaxN; topK, topP
// and minS, paper Sec. 3.1): two kernels per group of row tiles instead of the
// passes of select.hip.
//   k_short_scores  the pooled scores of up to 64 rows x `split` keys per
//                   workgroup, written to the workspace as fp32 (the products
//                   of the score passes, with the MFMA operands' roles swapped:
//                   a lane then holds one key of 16 rows, so a row's 32 keys go
//                   out as one 128-byte line; each score is the same sum in the
//                   same order, bit-identical to the passes').
//   k_short_select  one workgroup of W waves per row holds the row's scores in
//                   registers, finds the cut (rank, mass or threshold) and
//                   writes the ascending list.
// A long row must not be written to memory (75k tokens, 40 heads: 14 GB of
// scores against 1.5 GB of keys), but a short sequence's scores stay in the
// last-level cache, and the passes' 23 launches, most of them idle or waiting
// for the one before, cost more than they save; on many rows they save more,
// and launch_select takes them (passes_are_faster in select.hip).  Row tiles are
// taken in groups whose scores fit the workspace (at most kShortScoreBytes), one
// pair of launches per group.
#include <float.h>

#include <algorithm>
#include <type_traits>

#include "device_common.h"
#include "launch.h"
#include "select_common.h"

namespace vecattn {
namespace {

constexpr int kTileRows = 64;         // pooled rows per tile of k_short_scores
constexpr int kCandS = 128;           // keys ranked against one another at the end
// Scores of one group of row tiles: half the last-level cache, so that the
// second kernel reads them from there.
constexpr size_t kShortScoreBytes = size_t(128) << 20;
constexpr int64_t kShortManyRows = 4096;  // rows that fill the chip with one wave each

struct ShortParams {
  const uint16_t* qp;  // pooled queries [rows][D]
  const uint16_t* k;
  int64_t k_sB, k_sH, k_sN;
  float* s;            // scores of this group of tiles: [tiles * tile_rows][ld]
  int64_t ld;          // N rounded up to 32
  int64_t tile0, tiles;
  int tile_rows;       // rows a tile takes in s: 64, or N_p when a head has one tile
  int32_t* idx;
  int32_t* counts;
  int32_t* n_clamped;
  int64_t cap;
  int Hq, Hkv, group, N, P, Np, nrb, causal, keep_diag, unpadded, mode;
  int split, nsplit;   // keys per workgroup of k_short_scores
  int quads;           // lists start on 16 bytes
  float tau;
  double param;
  int per_head;
  double head_param[kMaxHeadParams];
};

// ---------------------------------------------------------------------------
// Scores.  64 keys at a time go into LDS (direct loads of whole rows, two
// stages, the attention's swizzle), and wave (half, kq) multiplies 32 of the
// tile's rows with 32 of them.  Loaded as MFMA operands instead (32 rows x 32
// bytes per instruction) K cost the address path four times as much: 22.2 us a
// launch at 12k tokens, and 28 with the rows split over two waves.  Bound by
// latency and, at 4k tokens and up, by the writes (4 bytes a score).
// ---------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(256) void k_short_scores(ShortParams p) {
  constexpr int DS = D / 16;
  constexpr int CH = D / 8;             // 16-byte chunks per row
  constexpr int U = 64 * CH / 256;      // direct loads per wave and stage
  __shared__ __align__(16) uint16_t k_s0[64 * D];
  __shared__ __align__(16) uint16_t k_s1[64 * D];
  const int64_t items = p.tiles * p.nsplit;
  const int64_t item = xcd_work_item((items + 7) / 8);
  if (item >= items) return;
  const int64_t t = item / p.nsplit;
  const int sp = static_cast<int>(item % p.nsplit);
  const int64_t tile = p.tile0 + t;
  const int rb = static_cast<int>(tile % p.nrb);
  const int64_t bh = tile / p.nrb;
  const int b = static_cast<int>(bh / p.Hq), h = static_cast<int>(bh % p.Hq);
  const int i0 = rb * kTileRows;
  const int nrows = min(kTileRows, p.Np - i0);
  const int Ltile = eligible(i0 + nrows - 1, p.P, p.N, p.causal);
  const int key0 = sp * p.split, key1 = min(key0 + p.split, Ltile);
  if (key0 >= key1) return;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, g = lane >> 5, ln = lane & 31;
  const int r0 = 32 * (wave & 1), c0 = 32 * (wave >> 1);
  const uint16_t* kh = p.k + b * p.k_sB + (h / p.group) * p.k_sH;
  auto kbuf = [&](int st) __attribute__((always_inline)) { return st ? k_s1 : k_s0; };
  auto issue = [&](int kb, int st) __attribute__((always_inline)) {
#if defined(__HIP_DEVICE_COMPILE__)
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int at = (wave * U + u) * 64 + lane;
      const int row = at / CH, col = (at % CH) ^ swz<D>(at / CH);
      const int64_t key = min(kb + row, p.N - 1);
      __builtin_amdgcn_global_load_lds(
          (const __attribute__((address_space(1))) void*)(kh + key * p.k_sN + 8 * col),
          LDS_PTR(void, kbuf(st) + (wave * U + u) * 64 * 8), 16, 0, 0);
    }
#endif
  };
  issue(key0, 0);
  // A operand: pooled row r0 + ln, head-dim slots 16 s2 + 8 g .. +7.
  bf16x8 qf[DS];
  {
    const int rl = r0 + ln;
    const u32x4* src = reinterpret_cast<const u32x4*>(
        p.qp + (bh * p.Np + i0 + (rl < nrows ? rl : 0)) * D);
#pragma unroll
    for (int s2 = 0; s2 < DS; ++s2) {
      const u32x4 w = rl < nrows ? src[2 * s2 + g] : u32x4{0, 0, 0, 0};
      qf[s2] = __builtin_bit_cast(bf16x8, w);
    }
  }
  // Stores through a buffer resource over these rows: one lane offset, the
  // row's as a scalar (a tile's rows span < 2^23 bytes).
  const int ld4 = static_cast<int>(p.ld) * 4;
  const int left = nrows - r0;
  const __amdgpu_buffer_rsrc_t out = __builtin_amdgcn_make_buffer_rsrc(
      p.s + (t * p.tile_rows + r0) * p.ld, 0, max(min(left, 32), 0) * ld4, 0x00020000);
  const int voff = 4 * g * ld4 + 4 * ln;
  auto step = [&](int kb, int st) __attribute__((always_inline)) {
    wait_vmcnt<0>();
    __builtin_amdgcn_s_barrier();  // this stage has landed, the other one has been read
    if (kb + 64 < key1) issue(kb + 64, st ^ 1);
    if (left <= 0 || kb + c0 >= key1) return;
    const char* kr = reinterpret_cast<const char*>(kbuf(st)) + (c0 + ln) * 2 * D;
    u32x4 kf[DS];
#pragma unroll
    for (int s2 = 0; s2 < DS; ++s2)
      kf[s2] = *reinterpret_cast<const u32x4*>(kr + 16 * ((2 * s2 + g) ^ swz<D>(c0 + ln)));
    f32x16 acc = f32x16{};
#pragma unroll
    for (int s2 = 0; s2 < DS; ++s2)
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf[s2], __builtin_bit_cast(bf16x8, kf[s2]), acc,
                                                    0, 0, 0);
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int rl = 8 * (v / 4) + v % 4;
      if (left >= 32 || rl + 4 * g < left)
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(acc[v]), out, voff + 4 * (kb + c0),
                                              rl * ld4, 0);
    }
  };
  for (int kb = key0; kb < key1; kb += 128) {
    step(kb, 0);
    if (kb + 64 < key1) step(kb + 64, 1);
  }
}

// ---------------------------------------------------------------------------
// The cut and the list of one row.  A lane holds 4 * E4 scores, wave w the keys
// [w * E4 * 256, + E4 * 256) of the row (groups of 256 keys, 4 consecutive ones
// per lane); scores are clamped to finite floats (NaN: the lowest), ineligible
// keys are -inf.  The kept set is {score > tf} plus the keys scoring tf, all of
// them or those up to index it.
//   histogram  of the interval [flo, fhi] that holds the cut (at first all
//              keys), linear in the score the first time, in the ordered key,
//              by a shift, afterwards (each narrows the interval by the number
//              of bins, so at most 5), and the bin with the cut;
//   collect    that bin's keys: at most kCandS of them are ranked by (score
//              descending, index ascending) and the cut is one of them; else
//              their smallest and largest score are the next interval.
// topP: a bin carries its softmax mass (terms exp(tau (s - max)) <= 1, in units
// of 2^-31) besides its count; the bin chosen by those sums is checked against
// the fp64 sums of the terms above and inside it, and moved if they disagree.
// Bound by instruction issue: ~20 per key in four passes (load, histogram,
// collect, list); the passes handle the one group that may hold ineligible keys
// apart (4096 tokens, 28 heads, topK: 39.8 -> 36.8 us).  A lane holds few keys (16, or 32 past 8192) and a row takes
// more waves instead: with 64 keys per lane the unrolled passes spilled and
// outgrew the instruction cache (288 us for 2700 rows of 12k tokens).
// ---------------------------------------------------------------------------
// Waves per SIMD the registers must leave room for.  A row of 8 waves puts two
// on each SIMD, so 129 to 256 registers hold a CU to one row at a time: 28
// heads, 12345 tokens, topK 15% 368 us with 136 registers, 276 with 128 (two
// rows; 20 spilled), topP 575 us with 204, 520 with 128 (182 spilled); 7000
// tokens 93 -> 82 (80 registers, three rows), topP 201 -> 147 (128, two).  The
// four waves of a shorter row do without: 4096 tokens 36.5 us, 39.3 held to 64
// registers, topP 51.7 and 53.5 held to 96.
template <int W, int E4, bool TOPP>
constexpr int kSelectWaves = W < 8 ? 1 : E4 == 8 || TOPP ? 4 : 6;

template <int W, int E4, bool TOPP>
__global__ __launch_bounds__(64 * W)
    __attribute__((amdgpu_waves_per_eu(kSelectWaves<W, E4, TOPP>))) void k_short_select(ShortParams p) {
  constexpr int kWaveKeys = 256 * E4;
  constexpr int kBinsS = W >= 8 ? 1024 : 256;  // bins of one histogram
  constexpr int kLaneBins = kBinsS / 64;
  const int64_t t = blockIdx.x / p.tile_rows;
  const int rl = static_cast<int>(blockIdx.x % p.tile_rows);
  const int64_t tile = p.tile0 + t;
  const int i = static_cast<int>(tile % p.nrb) * kTileRows + rl;
  const int64_t bh = tile / p.nrb;
  if (i >= p.Np) return;
  const int64_t row = bh * p.Np + i;
  const int L = eligible(i, p.P, p.N, p.causal);
  const double prm = p.per_head ? p.head_param[bh % p.Hq] : p.param;

  using Bin = std::conditional_t<TOPP, unsigned long long, uint32_t>;  // topP: count << 48 | mass
  __shared__ Bin s_bins[kBinsS];
  __shared__ uint64_t s_cand[kCandS], s_sorted[kCandS];
  __shared__ uint32_t s_ncand;
  __shared__ uint32_t s_ru[2][W];
  __shared__ double s_rd[2][W];
  __shared__ __align__(16) uint16_t s_list[kWaveKeys * W];

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  auto sync = [&]() __attribute__((always_inline)) {
    if (W == 1) wave_sync();
    else __syncthreads();
  };
  // Reductions over the row's workgroup, uniform results.  Two slots taken in
  // turn: a slot is written again only after another barrier.
  int turn = 0;
  auto reduce_u32 = [&](uint32_t x, auto op) __attribute__((always_inline)) {
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) x = op(x, static_cast<uint32_t>(__shfl_xor(static_cast<int>(x), o)));
    if (W > 1) {
      if (lane == 0) s_ru[turn][wave] = x;
      __syncthreads();
      x = s_ru[turn][0];
#pragma unroll
      for (int w = 1; w < W; ++w) x = op(x, s_ru[turn][w]);
      turn ^= 1;
    }
    return static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(x)));
  };
  auto reduce_sum = [&](double x) __attribute__((always_inline)) {
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) x += __shfl_xor(x, o);
    if (W > 1) {
      if (lane == 0) s_rd[turn][wave] = x;
      __syncthreads();
      x = s_rd[turn][0];
#pragma unroll
      for (int w = 1; w < W; ++w) x += s_rd[turn][w];
      turn ^= 1;
    }
    return x;
  };
  auto umax = [](uint32_t a, uint32_t b) { return max(a, b); };
  auto umin = [](uint32_t a, uint32_t b) { return min(a, b); };
  auto uadd = [](uint32_t a, uint32_t b) { return a + b; };

  // Score e = 4 j + c of the lane is key pos(j) + c; the wave holds eligible
  // keys in its first `ng` groups.
  auto pos = [&](int j) __attribute__((always_inline)) { return wave * kWaveKeys + (j * 64 + lane) * 4; };
  const int ng = min(max((L - wave * kWaveKeys + 255) / 256, 0), E4);
  // Every key of group j is eligible (uniform: all groups but one or none).
  auto full = [&](int j) __attribute__((always_inline)) { return wave * kWaveKeys + (j + 1) * 256 <= L; };
  float f[4 * E4];
  float fmx = -FLT_MAX, fmn = FLT_MAX;
  {
    const float* src = p.s + (t * p.tile_rows + rl) * p.ld;
    f32x4 x[E4];
#pragma unroll
    for (int j = 0; j < E4; ++j)  // ld is a multiple of 4: a quad with an eligible key lies in the row
      x[j] = pos(j) < L ? *reinterpret_cast<const f32x4*>(src + pos(j)) : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int j = 0; j < E4; ++j) {
      if (full(j)) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          f[4 * j + c] = __builtin_amdgcn_fmed3f(x[j][c], -FLT_MAX, FLT_MAX);  // NaN: the lower bound
          fmx = fmaxf(fmx, f[4 * j + c]);
          fmn = fminf(fmn, f[4 * j + c]);
        }
      } else {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const float y = fminf(fmaxf(x[j][c], -FLT_MAX), FLT_MAX);
          const bool ok = pos(j) + c < L;
          f[4 * j + c] = ok ? y : kNegInf;
          fmx = fmaxf(fmx, f[4 * j + c]);
          fmn = fminf(fmn, ok ? y : FLT_MAX);
        }
      }
    }
  }
  // Makes the scores opaque, at the start of a pass over them: otherwise their
  // keys, terms and bins are kept in registers from pass to pass.
  auto touch = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int e = 0; e < 4 * E4; ++e) asm volatile("" : "+v"(f[e]));
  };
  const float mx = ord_val(reduce_u32(ord_key(fmx), umax));
  const float mn = ord_val(reduce_u32(ord_key(fmn), umin));

  const float tl2 = p.tau * 1.4426950408889634f;
  auto term = [&](float x) __attribute__((always_inline)) {  // softmax term (0 if ineligible)
    return __builtin_amdgcn_exp2f((x - mx) * tl2);
  };

  float tf = -FLT_MAX;       // keep scores > tf, and those equal to tf: all, or up to index it
  int it = 0x7FFFFFFF;
  bool some = false;         // only some of the keys scoring tf are kept
  bool clamped = false;
  bool by_mass = TOPP && prm < 1.0;  // p = 1 keeps every eligible key
  int want = L;
  double target = 0.0;       // mass to reach
  bool search = true;
  if (p.mode == kModeTopK) {
    want = topk_count(prm, L);
  } else if (p.mode == kModeMinS) {
    // s >= max - alpha / tau, rounded down so that keys at it are kept
    const double thr = static_cast<double>(mx) - prm / static_cast<double>(p.tau);
    float lo = static_cast<float>(thr);
    if (static_cast<double>(lo) > thr) lo = ord_val(ord_key(lo) - 1u);
    lo = fmaxf(lo, -FLT_MAX);
    uint32_t n = 0;
    touch();
#pragma unroll
    for (int e = 0; e < 4 * E4; ++e) n += f[e] >= lo ? 1u : 0u;
    if (static_cast<int64_t>(reduce_u32(n, uadd)) > p.cap) {
      want = static_cast<int>(p.cap);
      clamped = true;
    } else {
      tf = lo;
      search = false;
    }
  } else if (by_mass) {
    double z = 0.0;
    touch();
#pragma unroll
    for (int e = 0; e < 4 * E4; ++e) z += static_cast<double>(term(f[e]));
    target = prm * reduce_sum(z);
  } else if (TOPP && L > p.cap) {  // p = 1: the cap best of all keys
    want = static_cast<int>(p.cap);
    clamped = true;
  }
  if (!by_mass && want >= L) search = false;  // every eligible key
  while (search) {
    search = false;
    float flo = mn, fhi = mx;
    int inside = L, above = 0;     // keys in the interval (or its bin `cut`) and above it
    double m_above = 0.0;          // mass above it
    for (int level = 0; flo != fhi; ++level) {
      // First histogram: bin = floor(score * mul + add), clamped.  topP: the
      // mass lies within kTopPRange nats of the maximum; keys below that share
      // bin 0.  A range too small or large for finite factors puts every key
      // into bin 0 (mul = 0) and leaves the work to the next histogram; an
      // ineligible key (-inf, or NaN after mul = 0) also falls there.
      const float base = by_mass ? fmaxf(flo, fhi - kTopPRange / p.tau) : flo;
      float mul = static_cast<float>(kBinsS) / (fhi - base);
      if (!(mul < 1e30f)) mul = 0.0f;
      const float add = -base * mul;
      constexpr int kBits = kBinsS == 1024 ? 10 : 8;
      const uint32_t olo = ord_key(flo), ohi = ord_key(fhi);
      const int sh = max(0, 32 - kBits - static_cast<int>(__builtin_clz(ohi - olo)));
      auto bin0 = [&](float x) __attribute__((always_inline)) {
        return static_cast<int>(__builtin_amdgcn_fmed3f(__builtin_fmaf(x, mul, add), 0.0f,
                                                        static_cast<float>(kBinsS - 1)));
      };
      auto bin1 = [&](float x) __attribute__((always_inline)) {
        return static_cast<int>((ord_key(x) - olo) >> sh);
      };
      auto entry = [&](float x) __attribute__((always_inline)) {
        if constexpr (TOPP)
          return (1ull << 48) | (by_mass ? static_cast<uint32_t>(__builtin_fmaf(term(x), 0x1p31f, 0.5f)) : 0u);
        else
          return 1u;
      };
      int cut = -1;  // -1: every key of the interval
      if (inside > kCandS) {
        for (int b = tid; b < kBinsS; b += 64 * W) s_bins[b] = 0;
        sync();
        touch();
        if (level == 0) {
#pragma unroll
          for (int j = 0; j < E4; ++j) {
            if (j >= ng) break;
#pragma unroll
            for (int c = 0; c < 4; ++c) {  // an ineligible key counts in bin 0 (taken off below)
              const float x = f[4 * j + c];
              atomicAdd(&s_bins[bin0(x)], entry(x));
            }
          }
        } else {
#pragma unroll
          for (int e = 0; e < 4 * E4; ++e)
            if (f[e] >= flo && f[e] <= fhi) atomicAdd(&s_bins[bin1(f[e])], entry(f[e]));
        }
        sync();
        if (level == 0 && tid == 0) {
          // eligible keys fill whole groups but the last one
          const int extra = (L + 255) / 256 * 256 - L;
          if constexpr (TOPP) s_bins[0] -= static_cast<unsigned long long>(extra) << 48;
          else s_bins[0] -= static_cast<uint32_t>(extra);
        }
        sync();
        // Every wave alike: lane l holds kLaneBins bins from the top, bin
        // kBinsS - 1 - kLaneBins l - j.
        const Bin* mine = s_bins + (kBinsS - 1 - kLaneBins * lane);
        auto pick = [&](auto scan, auto weight, auto need) __attribute__((always_inline)) {
          decltype(weight(0)) sum = 0;
#pragma unroll
          for (int j = 0; j < kLaneBins; ++j) sum += weight(j);
          const auto incl = scan(sum);
          const uint64_t hit = __ballot(incl >= need);
          const int src = hit ? __builtin_ctzll(hit) : 63;
          auto upto = incl - sum;
          int jb = kLaneBins - 1;
          auto before = upto;
          bool found = false;
#pragma unroll
          for (int j = 0; j < kLaneBins; ++j) {
            const auto w = weight(j);
            if (!found) {
              before = upto;
              jb = j;
              found = upto + w >= need;
            }
            upto += w;
          }
          cut = __builtin_amdgcn_readlane(kBinsS - 1 - kLaneBins * lane - jb, src);
          if (!by_mass) {  // exact counts
            above += __builtin_amdgcn_readlane(static_cast<int>(before), src);
            inside = __builtin_amdgcn_readlane(static_cast<int>(weight(jb)), src);
          }
        };
        if (TOPP && by_mass) {
          pick([](uint64_t x) { return wave_scan(x); },
               [&](int j) -> uint64_t { return mine[-j] & ((1ull << 48) - 1ull); },
               static_cast<uint64_t>(fmax(ceil((target - m_above) * 0x1p31), 0.0)));
        } else {
          pick([](int x) { return wave_incl_scan(x); },
               [&](int j) -> int { return static_cast<int>(TOPP ? static_cast<uint64_t>(mine[-j]) >> 48 : mine[-j]); },
               want - above);
        }
      }
      float lo, hi;
      int dir = 0;
      for (;;) {
        sync();  // s_ncand and s_cand of the pass before have been read
        if (tid == 0) s_ncand = 0u;
        sync();
        lo = FLT_MAX;
        hi = -FLT_MAX;
        uint32_t nab = 0;
        double m_in = 0.0, m_ab = 0.0;
        auto member = [&](int e) __attribute__((always_inline)) {
          lo = fminf(lo, f[e]);
          hi = fmaxf(hi, f[e]);
          const uint32_t at = atomicAdd(&s_ncand, 1u);
          if (at < kCandS)
            s_cand[at] = (static_cast<uint64_t>(ord_key(f[e])) << 32) |
                         ~static_cast<uint32_t>(pos(e / 4) + e % 4);
          if (TOPP && by_mass) m_in += static_cast<double>(term(f[e]));
        };
        touch();
        if (level == 0 && cut >= 0) {
#pragma unroll
          for (int j = 0; j < E4; ++j) {
            if (j >= ng) break;
            int bn[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) bn[c] = bin0(f[4 * j + c]);
            if (!full(j)) {
#pragma unroll
              for (int c = 0; c < 4; ++c) bn[c] = f[4 * j + c] == kNegInf ? -1 : bn[c];
            }
            if (bn[0] == cut || bn[1] == cut || bn[2] == cut || bn[3] == cut) {
#pragma unroll
              for (int c = 0; c < 4; ++c)
                if (bn[c] == cut) member(4 * j + c);
            }
            if (TOPP && by_mass) {
#pragma unroll
              for (int c = 0; c < 4; ++c) {
                nab += bn[c] > cut ? 1u : 0u;
                m_ab += bn[c] > cut ? static_cast<double>(term(f[4 * j + c])) : 0.0;
              }
            }
          }
        } else {
#pragma unroll
          for (int e = 0; e < 4 * E4; ++e) {
            if (!(f[e] >= flo && f[e] <= fhi)) continue;
            const int bn = cut < 0 ? -1 : bin1(f[e]);
            if (bn == cut) {
              member(e);
            } else if (TOPP && by_mass && bn > cut) {
              ++nab;
              m_ab += static_cast<double>(term(f[e]));
            }
          }
        }
        sync();
        if (TOPP && by_mass && cut >= 0) {
          // The masses in fp64, and a neighbouring bin if they rule this one
          // out: up while the bins above reach the target without it, down
          // while it falls short (never past the interval's last key).
          const int nin = static_cast<int>(s_ncand);
          const int n_ab = static_cast<int>(reduce_u32(nab, uadd));
          m_in = reduce_sum(m_in);
          m_ab = m_above + reduce_sum(m_ab);
          if (m_ab >= target && dir <= 0 && n_ab > 0) {
            dir = -1;
            ++cut;
            continue;
          }
          if ((m_ab + m_in < target || nin == 0) && cut > 0 && nin + n_ab < inside) {
            dir = 1;
            --cut;
            continue;
          }
          m_above = m_ab;
          above += n_ab;
          inside = nin;
        }
        break;
      }
      if (inside <= kCandS) break;
      flo = ord_val(reduce_u32(ord_key(lo), umin));
      fhi = ord_val(reduce_u32(ord_key(hi), umax));
    }
    int count;
    if (flo == fhi) {  // one score: the first `n` of its keys by index
      int n = want - above;
      if (TOPP && by_mass) {
        const double m = static_cast<double>(term(flo));
        const double need = m > 0.0 ? ceil((target - m_above) / m) : static_cast<double>(inside);
        n = static_cast<int>(fmin(fmax(need, 1.0), static_cast<double>(inside)));
      }
      n = min(max(n, 1), inside);
      count = above + n;
      tf = flo;
      some = n < inside;
      if (some) {  // smallest index with n of them up to it
        int a = -1, z = L - 1;
        while (z - a > 1) {
          const int m = a + (z - a) / 2;
          uint32_t c = 0;
          touch();
#pragma unroll
          for (int e = 0; e < 4 * E4; ++e) c += f[e] == flo && pos(e / 4) + e % 4 <= m ? 1u : 0u;
          if (static_cast<int>(reduce_u32(c, uadd)) >= n) z = m;
          else a = m;
        }
        it = z;
      }
    } else {  // rank the collected keys
      const int nc = min(inside, kCandS);
      for (int a = tid; a < nc; a += 64 * W) {
        const uint64_t mine = s_cand[a];
        int rank = 0;
#pragma unroll 4
        for (int b = 0; b < nc; ++b) rank += s_cand[b] > mine ? 1 : 0;
        s_sorted[rank] = mine;
      }
      sync();
      int n = want - above;
      if (TOPP && by_mass) {  // shortest prefix reaching the target; every wave alike
        const double ref = static_cast<double>(p.tau) * static_cast<double>(mx);
        double m[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const int a = 2 * lane + j;
          m[j] = a < nc ? mass_term(ord_val(static_cast<uint32_t>(s_sorted[a] >> 32)), p.tau, ref) : 0.0;
        }
        const double incl = wave_scan(m[0] + m[1]);
        const uint64_t hit = __ballot(m_above + incl >= target);
        const int src = hit ? __builtin_ctzll(hit) : 63;
        const int second = m_above + incl - m[1] >= target ? 0 : 1;
        n = hit ? __builtin_amdgcn_readlane(2 * lane + second + 1, src) : nc;
        if (target - m_above <= 0.0) n = 1;
      }
      n = min(max(n, 1), nc);
      const uint64_t last = n > 0 ? s_sorted[n - 1] : ~0ull;
      const uint32_t ot = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(last >> 32)));
      tf = ord_val(ot);
      it = __builtin_amdgcn_readfirstlane(static_cast<int>(~static_cast<uint32_t>(last)));
      some = n < nc && static_cast<uint32_t>(s_sorted[n] >> 32) == ot;
      count = above + n;
    }
    if (by_mass && count > p.cap) {  // keep the cap best
      by_mass = false;
      clamped = true;
      want = static_cast<int>(p.cap);
      it = 0x7FFFFFFF;
      search = true;
      sync();  // the ranked keys have been read
    }
  }
  if (clamped && tid == 0 && p.n_clamped) atomicAdd(p.n_clamped, 1);

  // The list: a kept key's place is the number of kept keys before it, from
  // the lane masks of its group's four compares (a prefix sum over the lanes'
  // counts took three times the instructions), then out of LDS in order, -1
  // behind.
  int total = 0;
  auto write_list = [&](auto kept) __attribute__((always_inline)) {
    int n = 0;
    touch();
#pragma unroll
    for (int j = 0; j < E4; ++j) {
      if (j >= ng) break;
#pragma unroll
      for (int c = 0; c < 4; ++c) n += __builtin_popcountll(__ballot(kept(j, c)));
    }
    int start = 0;
    total = n;
    if (W > 1) {
      if (lane == 0) s_ru[turn][wave] = static_cast<uint32_t>(n);
      __syncthreads();
      total = 0;
#pragma unroll
      for (int w = 0; w < W; ++w) {
        if (w < wave) start += static_cast<int>(s_ru[turn][w]);
        total += static_cast<int>(s_ru[turn][w]);
      }
      start = __builtin_amdgcn_readfirstlane(start);
      total = __builtin_amdgcn_readfirstlane(total);
    }
    touch();
#pragma unroll
    for (int j = 0; j < E4; ++j) {
      if (j >= ng) break;
      uint32_t at = static_cast<uint32_t>(start);
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const uint64_t m = __ballot(kept(j, c));
        at = __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(m >> 32),
                                       __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m), at));
        start += __builtin_popcountll(m);
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const bool k = kept(j, c);
        if (k) s_list[at] = static_cast<uint16_t>(pos(j) + c);
        at += k ? 1u : 0u;
      }
    }
  };
  if (!some && !p.keep_diag) {
    write_list([&](int j, int c) __attribute__((always_inline)) { return f[4 * j + c] >= tf; });
  } else {
    // The keys of the block's own rows, where they are asked for.
    const int dlo = p.keep_diag ? i * p.P : 0, dhi = p.keep_diag ? min(L, dlo + p.P) : 0;
    write_list([&](int j, int c) __attribute__((always_inline)) {
      const float x = f[4 * j + c];
      const int key = pos(j) + c;
      return (x > tf || (x == tf && (!some || key <= it))) || (key >= dlo && key < dhi);
    });
  }
  sync();
  total = min(total, static_cast<int>(min<int64_t>(p.cap, p.N)));
  int32_t* out = p.idx + row * p.cap;
  const int64_t end = p.unpadded ? total : p.cap;
  if (p.quads) {
    for (int64_t a = 4 * tid; a < end; a += 256 * W) {
      int4 v;
      v.x = a < total ? s_list[a] : -1;
      v.y = a + 1 < total ? s_list[a + 1] : -1;
      v.z = a + 2 < total ? s_list[a + 2] : -1;
      v.w = a + 3 < total ? s_list[a + 3] : -1;
      if (a + 3 < end) {
        *reinterpret_cast<int4*>(out + a) = v;
      } else {
        out[a] = v.x;
        if (a + 1 < end) out[a + 1] = v.y;
        if (a + 2 < end) out[a + 2] = v.z;
      }
    }
  } else {
    for (int64_t a = tid; a < end; a += 64 * W) out[a] = a < total ? s_list[a] : -1;
  }
  if (tid == 0) p.counts[row] = total;
}

inline size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

struct ShortSizes {
  int64_t Np, rows, nrb, tiles, ld;
  int tile_rows;
  size_t qp, tile_bytes;
};

ShortSizes short_sizes(int64_t B, int64_t Hq, int64_t N, int64_t D, int32_t P) {
  ShortSizes z{};
  z.Np = (N + P - 1) / P;
  z.rows = B * Hq * z.Np;
  z.nrb = (z.Np + kTileRows - 1) / kTileRows;
  z.tiles = B * Hq * z.nrb;
  z.ld = (N + 31) / 32 * 32;
  z.tile_rows = static_cast<int>(std::min<int64_t>(z.Np, kTileRows));
  z.qp = align256(static_cast<size_t>(z.rows) * D * 2);
  z.tile_bytes = static_cast<size_t>(z.tile_rows) * z.ld * 4;
  return z;
}

template <bool TOPP>
void select_rows(const ShortParams& p, int64_t rows, dim3 grid, hipStream_t stream) {
  auto run = [&](auto kernel, int waves) {
    hipLaunchKernelGGL(kernel, grid, dim3(64 * waves), 0, stream, p);
  };
  // Waves per row: 16 keys per lane (32 past 8192 keys, where a row would take
  // 16 waves); below 1024 keys one wave while the rows alone fill the chip (its
  // steps need no barrier), else four.
  if (p.N <= 1024) rows >= kShortManyRows ? run(k_short_select<1, 4, TOPP>, 1) : run(k_short_select<4, 1, TOPP>, 4);
  else if (p.N <= 4096) run(k_short_select<4, 4, TOPP>, 4);
  else if (p.N <= 8192) run(k_short_select<8, 4, TOPP>, 8);
  else run(k_short_select<8, 8, TOPP>, 8);
}

}  // namespace

bool short_select_ok(int64_t N, int32_t mode) { return mode != kModeMinSTiled && N <= kShortMaxN; }

size_t short_select_min_bytes(int64_t B, int64_t Hq, int64_t N, int64_t D, int32_t P) {
  const ShortSizes z = short_sizes(B, Hq, N, D, P);
  return z.qp + z.tile_bytes;
}

size_t short_select_bytes(int64_t B, int64_t Hq, int64_t N, int64_t D, int32_t P) {
  const ShortSizes z = short_sizes(B, Hq, N, D, P);
  const size_t group = std::max<size_t>(1, kShortScoreBytes / z.tile_bytes);
  return z.qp + std::min<size_t>(z.tiles, group) * z.tile_bytes;
}

hipError_t launch_select_short(const SelectArgs& a, hipStream_t stream) {
  const int64_t B = a.q.B, Hq = a.q.H, Hkv = a.k.H, N = a.q.N, D = a.q.D;
  const ShortSizes z = short_sizes(B, Hq, N, D, a.block);
  if (a.workspace_bytes < z.qp + z.tile_bytes) return hipErrorInvalidValue;
  char* ws = static_cast<char*>(a.workspace);
  ShortParams p{};
  p.qp = reinterpret_cast<const uint16_t*>(ws);
  p.k = static_cast<const uint16_t*>(a.k.ptr);
  p.k_sB = a.k.sB;
  p.k_sH = a.k.sH;
  p.k_sN = a.k.sN;
  p.s = reinterpret_cast<float*>(ws + z.qp);
  p.ld = z.ld;
  p.tile_rows = z.tile_rows;
  p.idx = a.idx;
  p.counts = a.counts;
  p.n_clamped = a.n_clamped;
  p.cap = a.cap;
  p.Hq = static_cast<int>(Hq);
  p.Hkv = static_cast<int>(Hkv);
  p.group = static_cast<int>(Hq / Hkv);
  p.N = static_cast<int>(N);
  p.P = a.block;
  p.Np = static_cast<int>(z.Np);
  p.nrb = static_cast<int>(z.nrb);
  p.causal = a.causal;
  p.keep_diag = a.keep_diag;
  p.unpadded = a.unpadded;
  p.mode = a.mode;
  p.quads = a.cap % 4 == 0 && reinterpret_cast<uintptr_t>(a.idx) % 16 == 0;
  p.tau = 1.0f / sqrtf(static_cast<float>(D));
  p.param = a.param;
  p.per_head = a.head_params != nullptr;
  if (p.per_head)
    for (int64_t h = 0; h < Hq; ++h) p.head_param[h] = a.head_params[h];

  hipError_t e = launch_pool(a.q, a.block, ws, Hq * z.Np * D, z.Np * D, D, stream);
  if (e != hipSuccess) return e;
  const size_t room = std::min(a.workspace_bytes - z.qp, std::max(kShortScoreBytes, z.tile_bytes));
  const int64_t group = std::max<int64_t>(1, static_cast<int64_t>(room / z.tile_bytes));
  for (int64_t t0 = 0; t0 < z.tiles; t0 += group) {
    p.tile0 = t0;
    p.tiles = std::min(group, z.tiles - t0);
    // Keys per workgroup: as few as make ~1024 workgroups, in units of the 128
    // that its four waves take at a time.
    const int64_t most = (N + 127) / 128;
    const int64_t ns = std::min(most, std::max<int64_t>(1, 1024 / p.tiles));
    p.split = static_cast<int>((most + ns - 1) / ns * 128);
    p.nsplit = static_cast<int>((N + p.split - 1) / p.split);
    const int64_t items = p.tiles * p.nsplit;
    const dim3 sgrid(static_cast<unsigned>((items + 7) / 8 * 8));
    if (D == 128) hipLaunchKernelGGL(k_short_scores<128>, sgrid, dim3(256), 0, stream, p);
    else hipLaunchKernelGGL(k_short_scores<64>, sgrid, dim3(256), 0, stream, p);
    const dim3 rgrid(static_cast<unsigned>(p.tiles * z.tile_rows));
    if (a.mode == kModeTopP) select_rows<true>(p, z.rows, rgrid, stream);
    else select_rows<false>(p, z.rows, rgrid, stream);
  }
  return hipGetLastError();
}

}  // namespace vecattn
