// Vector-sparse attention (paper Eq. 4, Sec. 3.2; appendix Algorithm 2) for gfx950.
//
// One workgroup owns up to 64 query rows (4 waves) or, for blocks of a
// multiple of 128 rows, up to 128 (8 waves) of one query block of one head and
// walks the block's index list I[b,h,i,0:C) in tiles of 64 keys
// (starting at the tile where the workgroups running on its XCD are, and
// wrapping around; see below).  Blocks are dealt to groups of XCDs sized so
// that the heads swept at once fit the last-level cache (xcd_group).
// The K and V rows of a tile are gathered straight from global memory into
// LDS (global_load_lds, 16 B per lane, no register staging) two tiles deep,
// stored row-major with an XOR swizzle of their 16-byte chunks so that both
// the row reads of K and the transposing reads of V (ds_read_b64_tr_b16) are
// free of bank conflicts.  The waves compute S^T = K_tile Q^T and
// O^T += V_tile^T P^T with v_mfma_f32_32x32x16_bf16 and keep the
// online-softmax state in registers.  Wave w = (rw, kw): rw picks 32 of the
// workgroup's query rows, kw picks 32 of the 64 keys of each tile; the two
// key halves are merged at the end.
//
// MFMA 32x32x16 lane layout (lane l, g = l / 32):
//   A (M x K): lane holds row l % 32, K-slots 8g .. 8g + 7
//   B (K x N): lane holds column l % 32, K-slots 8g .. 8g + 7
//   C (M x N): lane holds column l % 32, rows 8 * (v / 4) + 4g + v % 4, v < 16
// Only the pairing of K-slots between A and B matters for the product, so the
// keys of a K-step are ordered to match C's row order.
//
// ds_read_b64_tr_b16, per group of 16 lanes: lane 4p + c receives as element q
// the c-th 16-bit value at the address supplied by lane 4q + p.
#include <algorithm>
#include <type_traits>

#include "device_common.h"
#include "launch.h"

namespace vecattn {
namespace {

constexpr int kTile = 64;     // keys per gathered tile
// Progress of this kernel's workgroups on each XCD since the library was
// loaded, in units of 1/kHerdUnit of a list (wraps at 2^32).  It paces the
// tile order below: a locality hint only, so concurrent calls sharing it
// affect speed, never results.  Each XCD's counter has cache lines of its own:
// with all eight in one line the chip's updates serialised, ~21 ns each, which
// bounded launches of short lists (40 heads, 40 packed sequences of 700 tokens,
// two tiles a list: 701 us, 420 apart; 4 x 12 heads, 4096 tokens, 13 tiles: 104,
// 75; 24 heads, 24001 tokens, 75 tiles: 1545, 1509).
constexpr int kHerdStride = 64;
__device__ __align__(256) unsigned int g_herd[8 * kHerdStride];
constexpr int kHerdUnit = 4096;
// Tiles per update of that counter: updates to one address serialise in L2,
// so they must be rare next to the gathers.
constexpr int kHerdBatch = 16;

typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef short i16x8 __attribute__((ext_vector_type(8)));
// 16-byte copy per lane from a buffer (byte offset voff) to LDS (destination:
// wave-uniform base + 16 * lane).  The 16-byte form exists only on gfx950;
// the host pass of the compiler rejects it, so it is compiled for the device
// side only.
__device__ __forceinline__ void gather16_to_lds(__amdgpu_buffer_rsrc_t rsrc, uint32_t voff,
                                                void* lds_base) {
#if defined(__HIP_DEVICE_COMPILE__)
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, LDS_PTR(void, lds_base), 16, voff, 0, 0, 0);
#endif
}

// 4-byte copy per lane of a list entry to LDS through the list's buffer
// resource: offsets past the list read 0, so no index can leave the list.
__device__ __forceinline__ void ids_to_lds(__amdgpu_buffer_rsrc_t rsrc, uint32_t voff,
                                           void* lds_base) {
#if defined(__HIP_DEVICE_COMPILE__)
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, LDS_PTR(void, lds_base), 4, voff, 0, 0, 0);
#endif
}

// Lane u of each row of 16 lanes, to all lanes of that row (a DPP operand of
// the instruction that uses it).
template <int U>
__device__ __forceinline__ int row_bcast(int x) {
  return __builtin_amdgcn_update_dpp(0, x, 0x150 + U, 0xf, 0xf, true);
}

// The sequences of one launch over a packed batch, longest first: sequence s
// owns workgroups [end[s - 1], end[s]), a multiple of 8 of them, so that a
// workgroup's XCD is the same within its sequence as in the launch.
constexpr int kMaxSeqs = 32;
struct SeqTable {
  int32_t n;
  int32_t end[kMaxSeqs];
  int32_t row0[kMaxSeqs];    // first packed row
  int32_t len[kMaxSeqs];
  int32_t first[kMaxSeqs];   // query blocks of the sequences packed before it
  int32_t xgroup[kMaxSeqs];
};
struct OneSeq {};

// SAME_STRIDE: K and V rows have the same stride, so a gathered row's K and V
// offsets coincide.  ROWS: query rows per workgroup (64: 4 waves, or 128: 8
// waves, for blocks of a multiple of 128 rows, so that one gather of a tile
// serves all 128 rows of the block).  Held to two waves per SIMD (256
// registers): with one, nothing hides a wave's waits (dense keys, 64-row
// workgroups, 299 registers: 1.66 ms where two waves take 1.17).  SEQS: OneSeq,
// or the SeqTable of a packed batch (B = 1, no block order).
template <int D, bool SAME_STRIDE, int ROWS, typename SEQS>
__global__ __launch_bounds__(4 * ROWS) __attribute__((amdgpu_waves_per_eu(2))) void k_sparse_attn(
    const uint16_t* __restrict__ q, int64_t q_sB, int64_t q_sH, int64_t q_sN,
    const uint16_t* __restrict__ k, int64_t k_sB, int64_t k_sH, int64_t k_sN,
    const uint16_t* __restrict__ v, int64_t v_sB, int64_t v_sH, int64_t v_sN,
    uint16_t* __restrict__ o, int64_t o_sB, int64_t o_sH, int64_t o_sN, float* __restrict__ lse,
    const int32_t* __restrict__ idx, const int32_t* __restrict__ counts,
    const int32_t* __restrict__ order, int64_t cap, int32_t Hq,
    int32_t group, int32_t N, int32_t P, int32_t Np, int32_t chunks, int32_t causal,
    float scale_log2, int64_t total, int32_t xgroup, int32_t herd_slots, SEQS seqs) {
  constexpr int CH = D / 8;                 // 16-byte chunks per row
  constexpr int kThreads = 4 * ROWS;  // 2 key halves x ROWS / 32 row groups, 64 lanes each
  constexpr int RG = ROWS / 32;             // row groups (waves per key half)
  constexpr int U = kTile * CH / kThreads;  // direct-load instructions per wave per matrix
  constexpr int DS = D / 16;                // MFMA K-steps over the head dimension
  constexpr int DB = D / 32;                // 32-wide blocks of the head dimension
  constexpr int RB = 2 * D;                 // bytes per LDS row
  constexpr bool kPrio = ROWS == 64;         // raised priority for the MFMA bursts
  // Each pipeline stage is its own LDS object, so that the compiler can tell
  // that reads of one stage do not depend on the gathers in flight into the
  // other and does not make them wait for those.
  __shared__ __align__(16) uint16_t k_s0[kTile * D];
  __shared__ __align__(16) uint16_t k_s1[kTile * D];
  __shared__ __align__(16) uint16_t v_s0[kTile * D];
  __shared__ __align__(16) uint16_t v_s1[kTile * D];
  __shared__ __align__(16) int32_t id_s0[kTile];
  __shared__ __align__(16) int32_t id_s1[kTile];
  __shared__ float s_ml[RG][128];  // (m, l) of the kw = 1 waves for the merge
  // Stage selectors; always called with a constant stage, so they fold to a
  // direct reference to one LDS object.
  auto kbuf = [&](int st) __attribute__((always_inline)) { return st ? k_s1 : k_s0; };
  auto vbuf = [&](int st) __attribute__((always_inline)) { return st ? v_s1 : v_s0; };
  auto ibuf = [&](int st) __attribute__((always_inline)) { return st ? id_s1 : id_s0; };

  int bx = blockIdx.x;
  if constexpr (std::is_same_v<SEQS, SeqTable>) {
    int s = 0;
    while (s < seqs.n - 1 && bx >= seqs.end[s]) ++s;
    if (s > 0) bx -= seqs.end[s - 1];
    const int64_t r0 = seqs.row0[s];
    q += r0 * q_sN;
    k += r0 * k_sN;
    v += r0 * v_sN;
    o += r0 * o_sN;
    if (lse) lse += Hq * r0;
    const int64_t f0 = static_cast<int64_t>(seqs.first[s]) * Hq;
    idx += f0 * cap;
    counts += f0;
    N = seqs.len[s];
    Np = (N + P - 1) / P;
    total = static_cast<int64_t>(Hq) * Np * chunks;
    xgroup = seqs.xgroup[s];
  }

  // Work item: head bh = b * Hq + h, position pos in the head (block
  // order[bh, pos], or pos) and 64- or 128-row chunk of the block; the chunks
  // of a block stay on one XCD (they gather the same list).  XCDs form
  // 8 / xgroup groups.  Each group owns `whole` = nheads / groups whole heads,
  // in order, so that few heads are swept at once (their K/V rows then compete
  // less for the chip-wide last-level cache); the nheads % groups heads left
  // over are shared by all groups, group g taking the positions p = g (mod
  // groups) of each, so that every group gets the same work whatever the
  // blocks' list lengths (a head split at a group boundary would leave one
  // side with its longest lists).  A group's sequence is dealt to its XCDs
  // one block at a time, and each XCD walks its share in order.  The grid
  // covers the longest sequence (group 0's); every item is taken once.
  const int ngroups = 8 / xgroup;
  const int64_t nheads = total / (static_cast<int64_t>(Np) * chunks);
  const int64_t whole = nheads / ngroups;
  const int grp = (bx & 7) / xgroup;
  const int64_t slot = bx >> 3;
  const int chunk = static_cast<int>(slot % chunks);
  const int64_t e = (slot / chunks) * xgroup + (bx & 7) % xgroup;
  int64_t bh;
  int pos;
  if (e < whole * Np) {
    bh = grp * whole + e / Np;
    pos = static_cast<int>(e % Np);
  } else {
    const int64_t e2 = e - whole * Np;
    const int64_t ng = (Np - grp + ngroups - 1) / ngroups;  // positions = grp (mod groups)
    if (ng <= 0) return;
    bh = whole * ngroups + e2 / ng;
    if (bh >= nheads) return;
    pos = static_cast<int>((e2 % ng) * ngroups + grp);
  }
  // Without a block order a causal head is taken from its last block, the
  // longest list, so that the launch ends on short ones.
  const int i = order ? min(max(order[bh * Np + pos], 0), Np - 1) : causal ? Np - 1 - pos : pos;
  const int b = static_cast<int>(bh / Hq);
  const int h = static_cast<int>(bh % Hq);
  const int hk = h / group;

  const int row0 = i * P + chunk * ROWS;
  const int row_end = min(N, min(i * P + P, row0 + ROWS));
  // A valid list holds distinct keys of [0, N), so at most N of them; the
  // clamp keeps the tile arithmetic below in range for any counts.
  const int count = __builtin_amdgcn_readfirstlane(static_cast<int>(
      min<int64_t>(min<int64_t>(max(counts[bh * Np + i], 0), cap), N)));
  const int32_t* list = idx + (bh * Np + i) * cap;
  const int ntiles = (count + kTile - 1) / kTile;
  // Tile order.  A block's keys are random rows of the head's K/V, far more
  // than an XCD's L2 holds; the workgroups running together on an XCD share
  // L2 hits only if they gather from the same key range at the same time.
  // Lists are ascending, so the fraction of its list a workgroup has walked
  // is a position in key space (the same for lists of different lengths).
  // Every workgroup adds its progress, in 1/kHerdUnit of its list, to its
  // XCD's counter; that sum over the XCD's workgroup slots is the mean
  // position of the workgroups running there, and a new workgroup starts at
  // the tile at that fraction of its own list (then wraps around), so the
  // workgroups on an XCD sweep the keys together at their actual pace.  The
  // order of the tiles changes only the order of the softmax sums (results
  // can differ between runs within fp32 rounding).  Causal lists are walked
  // from their first tile instead: block i's list lies in [0, (i + 1) P), so a
  // fraction of it is a different key position for every block, while the
  // walks from key 0 of lists of like length (taken together by the block
  // order) stay together.
  const int xcd = bx & 7;  // the hardware deals workgroup x to XCD x % 8
  const bool herd = !causal;
  __shared__ int s_rot;
  __shared__ int s_redo;  // some wave's O or l is not finite after the first walk
  if (threadIdx.x == 0) s_redo = 0;
  if (threadIdx.x == 0 && !herd) s_rot = 0;
  if (threadIdx.x == 0 && herd) {
    const unsigned int progress =
        __hip_atomic_load(&g_herd[xcd * kHerdStride], __ATOMIC_RELAXED,
                          __HIP_MEMORY_SCOPE_AGENT);
    const unsigned int at = (progress / static_cast<unsigned int>(herd_slots)) % kHerdUnit;
    // ntiles <= 2^18 (count <= N < 2^24), so the product fits 32 bits.
    s_rot = static_cast<int>((at * static_cast<unsigned int>(ntiles)) / kHerdUnit);
  }
  __syncthreads();
  const int t_rot = __builtin_amdgcn_readfirstlane(s_rot);
  // Progress after t tiles, in 1/kHerdUnit of the list (a whole list adds up
  // to kHerdUnit exactly).
  auto herd_units = [&](int t) __attribute__((always_inline)) {
    return static_cast<unsigned int>((kHerdUnit * t) / ntiles);
  };
  auto tile_of = [&](int t) __attribute__((always_inline)) {  // t-th tile processed
    if (t >= ntiles) return t;  // past the list (reads 0)
    const int x = t + t_rot;
    return x >= ntiles ? x - ntiles : x;
  };
  // The list entries of tile t as a buffer resource (scalar work only, so
  // that per-lane offsets stay loop-invariant); reads past the list return 0.
  auto tile_rsrc = [&](int t) __attribute__((always_inline)) {
    const int e0 = tile_of(t) * kTile;
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t*>(list) + e0, 0,
                                             max(count - e0, 0) * 4, 0x00020000);
  };

  // K and V of this head as buffer resources: gathers use 32-bit byte offsets
  // (row * row_bytes + 16 * chunk, the product in 24 bits); the host rejects
  // heads with N >= 2^24, a row stride of 2^24 bytes or more, or rows spanning
  // 2^31 bytes or more, so every offset here is exact.
  const uint16_t* kh = k + b * k_sB + hk * k_sH;
  const uint16_t* vh = v + b * v_sB + hk * v_sH;
  const uint32_t k_rowb = static_cast<uint32_t>(k_sN) * 2u;
  const uint32_t v_rowb = static_cast<uint32_t>(v_sN) * 2u;
  const __amdgpu_buffer_rsrc_t krs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(kh), 0, static_cast<int>((N - 1) * k_rowb + RB), 0x00020000);
  const __amdgpu_buffer_rsrc_t vrs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(vh), 0, static_cast<int>((N - 1) * v_rowb + RB), 0x00020000);

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  const int g = lane >> 5;
  const int ln = lane & 31;
  const int rw = wave % RG;
  const int kw = wave / RG;

  // Gather mapping: direct-load instruction u of this wave covers LDS chunks
  // [(wave*U + u)*64, +64) of a tile; lane -> (row r, physical chunk x), and
  // it fetches logical chunk x ^ swz(r) of key row ids[r].
  auto grow = [&](int u) __attribute__((always_inline)) { return ((wave * U + u) * 64 + lane) / CH; };
  auto gcol = [&](int u) __attribute__((always_inline)) {
    const int L = (wave * U + u) * 64 + lane;
    return (L % CH) ^ swz<D>(L / CH);
  };
  // Key ids of the next tile to gather (raw; clamped when used).  With
  // 16-chunk rows (D = 128) a row's 16 lanes are one DPP row, so one load
  // brings all U ids of the lane (lane u of a DPP row holds the id of
  // instruction u) and the gather's offset reads its own with a DPP
  // broadcast: U - 1 fewer vector-memory instructions per wave and tile.
  constexpr bool kRowIds = CH == 16 && U <= 4;
  constexpr int kIdRegs = kRowIds ? 1 : U;
  int nid[kIdRegs];

  auto load_ids = [&](int t) __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t rs = tile_rsrc(t);
    if constexpr (kRowIds) {
      const int row = (wave * U + (lane & (U - 1))) * 4 + (lane >> 4);
      nid[0] = __builtin_amdgcn_raw_buffer_load_b32(rs, row * 4, 0, 0);
    } else {
#pragma unroll
      for (int u = 0; u < U; ++u) nid[u] = __builtin_amdgcn_raw_buffer_load_b32(rs, grow(u) * 4, 0, 0);
    }
  };
  auto id_of = [&](int u) __attribute__((always_inline)) {
    if constexpr (kRowIds) {
      return u == 0 ? row_bcast<0>(nid[0]) : u == 1 ? row_bcast<1>(nid[0])
             : u == 2 ? row_bcast<2>(nid[0]) : row_bcast<3>(nid[0]);
    } else {
      return nid[u];
    }
  };
  // Gather n of the 2 U of a tile: the K rows of instruction n / 2, then its V
  // rows.  Valid ids are below N < 2^24 and row strides below 2^24 bytes, as
  // __umul24 needs; an invalid id reads some row of this head or zeros, never
  // outside it (buffer range check).
  auto gather = [&](int n, int st) __attribute__((always_inline)) {
    const int u = n / 2;
    const uint32_t r = static_cast<uint32_t>(id_of(u));
    if (n % 2 == 0) {
      gather16_to_lds(krs, __umul24(r, k_rowb) + 16u * gcol(u), kbuf(st) + (wave * U + u) * 64 * 8);
    } else {
      gather16_to_lds(vrs, __umul24(r, SAME_STRIDE ? k_rowb : v_rowb) + 16u * gcol(u),
                      vbuf(st) + (wave * U + u) * 64 * 8);
    }
  };
  auto stage_ids = [&](int t, int st) __attribute__((always_inline)) {
    if (wave == 0)  // the tile's key ids (past count: 0, and masked)
      ids_to_lds(tile_rsrc(t), static_cast<uint32_t>(lane) * 4u, ibuf(st));
  };

  // Q^T operand: this lane's query row, head-dim slots 16s + 8g .. +7.  The first
  // tile's ids are on their way already, and its gathers follow as soon as they
  // are here: the first step's wait covers Q as well, where Q, ids and gathers
  // one after another cost a list of two tiles 4% (28 heads, 8192 tokens, causal,
  // 1% of the keys: 62.0 -> 59.5 us; 10%: 106, 102).
  if (ntiles > 0) load_ids(0);
  const int my_row = row0 + 32 * rw + ln;
  bf16x8 qf[DS];
  {
    const bool have = my_row < row_end;
    const u32x4* qr = reinterpret_cast<const u32x4*>(
        q + b * q_sB + h * q_sH + static_cast<int64_t>(have ? my_row : row0) * q_sN);
#pragma unroll
    for (int s = 0; s < DS; ++s) {
      const u32x4 t = have ? qr[2 * s + g] : u32x4{0, 0, 0, 0};
      qf[s] = __builtin_bit_cast(bf16x8, t);
    }
  }

  f32x16 oacc[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db) oacc[db] = f32x16{};
  // Reference (log2 units) this lane's row is scaled against; kUnseen until the
  // row has met a visible key.
  constexpr float kUnseen = -3.4028234663852886e38f;
  float m_run = kUnseen;
  float l_run = 0.0f;   // this lane's partial normaliser
  int settled = 0;      // every row of the wave has a reference
  float lim = 256.0f;   // a tile sum above it moves references after the weights
  int careful = 0;      // second walk: references are fixed before the weights
  int moved = 0;        // some tile of this wave had weights above 256

  // Per-lane byte offsets of the LDS reads inside a stage, opaque to the
  // compiler so that each stage's address is a constant offset from them (one
  // register per offset for all stages, not one per stage).
  const int j16 = lane & 15;
  const int tq = j16 >> 2, tp = j16 & 3;
  const int vhalf = (lane >> 4) & 1;
  uint32_t koff[DS], voff[DB][2];
#pragma unroll
  for (int s2 = 0; s2 < DS; ++s2) {
    const int krow = 32 * kw + ln;
    koff[s2] = krow * RB + 16 * ((2 * s2 + g) ^ swz<D>(krow));
    asm volatile("" : "+v"(koff[s2]));
  }
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int hi = 0; hi < 2; ++hi) {
      const int d = 32 * db + 16 * vhalf + 4 * tp;   // first of the 4 head-dim values addressed
      const int k0 = 32 * kw + 4 * g + tq + 8 * hi;  // key row this lane addresses (K-step 0)
      voff[db][hi] = k0 * RB + 16 * ((d >> 3) ^ swz<D>(k0)) + 8 * ((d >> 2) & 1);
      asm volatile("" : "+v"(voff[db][hi]));
    }

  // One tile.  MORE: tile t + 1 exists and is gathered meanwhile.
  auto step = [&](const int t, const int st, auto more_tag) __attribute__((always_inline)) {
    constexpr bool MORE = decltype(more_tag)::value;
    // Tile t has landed, and the ids of tile t+1 (issued right after it) too;
    // the barrier (no fence: all LDS traffic here is waited for explicitly)
    // also guarantees every wave is done reading the other stage.
    wait_vmcnt<0>();
    __builtin_amdgcn_s_barrier();
    if (herd && !careful && wave == 0 && lane == 0 && (t % kHerdBatch) == kHerdBatch - 1)
      __hip_atomic_fetch_add(&g_herd[xcd * kHerdStride],
                             herd_units(t + 1) - herd_units(t + 1 - kHerdBatch), __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
    if (MORE) stage_ids(t + 1, st ^ 1);

    // S^T = K_tile Q^T for this wave's 32 keys x 32 rows, and between its MFMAs
    // the gathers of tile t + 1.  A gather holds the CU's address path 16
    // cycles (1 KB at 64 B per cycle) and a wave that issues while the path is
    // full waits; the workgroup's gathers issued in one burst before the MFMAs
    // cost the step those ~512 cycles (2155 cycles per tile with two workgroups
    // on a CU, 1521 with the tiles resident), one per MFMA runs them beside the
    // matrix pipe (1842; 75k DiT layer 5.29 -> 4.87 ms per 10 heads, 119k DiT
    // 14.5 -> 13.7 per 6).  Issued any later (softmax, P V) they land late:
    // 2374 cycles.
    const char* kb = reinterpret_cast<const char*>(kbuf(st));
    u32x4 kf[DS];
#pragma unroll
    for (int s2 = 0; s2 < DS; ++s2) kf[s2] = *reinterpret_cast<const u32x4*>(kb + koff[s2]);
    f32x16 sacc = f32x16{};
    // In 64-row workgroups the score MFMAs run at raised wave priority, so that
    // a wave issuing them is not held back by the softmax work of the other
    // wave on its SIMD (which belongs to the other workgroup, at another point
    // of its step).  The two waves a SIMD holds of an 8-wave workgroup are at
    // the same point of the same step, and do as well without it.
    if (kPrio) __builtin_amdgcn_s_setprio(2);
#pragma unroll
    for (int s2 = 0; s2 < DS; ++s2) {
      sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kf[s2]), qf[s2], sacc,
                                                     0, 0, 0);
      if (MORE) {
        static_assert(2 * U <= DS, "at most one gather per score MFMA");
        if (s2 % (DS / (2 * U)) == 0) {
          const int n = s2 / (DS / (2 * U));
          __builtin_amdgcn_sched_barrier(0);
          gather(n, st ^ 1);
          if (n == 2 * U - 1) load_ids(t + 2);  // past the list these read 0
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    if (kPrio) __builtin_amdgcn_s_setprio(0);
    // The V^T operands (transposing LDS reads) are fetched now, so that their
    // latency hides behind the score MFMAs and the softmax.
    const char* vb = reinterpret_cast<const char*>(vbuf(st));
    auto vread = [&](int ks, uint32_t o0, uint32_t o1) __attribute__((always_inline)) {
      const char* a0 = vb + o0 + 16 * ks * RB;  // the swizzle repeats every 16 rows
      const char* a1 = vb + o1 + 16 * ks * RB;
      const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(i16x4, a0));
      const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(i16x4, a1));
      return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    bf16x8 vfrag[DB][2];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) vfrag[db][ks] = vread(ks, voff[db][0], voff[db][1]);

    // Masks are needed only on the list's last tile and, when causal, on tiles
    // reaching past this wave's first row (lists are ascending).
    const int tbase = tile_of(t) * kTile;
    const int nvalid = min(kTile, count - tbase);
    const int32_t* ids = ibuf(st);
    if (nvalid < kTile ||
        (causal && __builtin_amdgcn_readfirstlane(ids[nvalid - 1]) > row0 + 32 * rw)) {
#pragma unroll
      for (int m4 = 0; m4 < 4; ++m4) {
        const int kl = 32 * kw + 8 * m4 + 4 * g;
        const int lim = nvalid - kl;  // entries e < lim of this group are in the list
        const int4 jj = *reinterpret_cast<const int4*>(ids + kl);
        const int js[4] = {jj.x, jj.y, jj.z, jj.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const bool ok = (e < lim) && (!causal || js[e] <= my_row);
          sacc[4 * m4 + e] = ok ? sacc[4 * m4 + e] : kNegInf;
        }
      }
    }
    // References.  Until every row of the wave has met a visible key (usually
    // after the first tile), and throughout a careful walk, rows whose maximum
    // grew by more than 8 (log2 units) move their reference before the weights
    // are computed, and O and l are rescaled.
    if (!settled) {
      float tmax = kNegInf;
#pragma unroll
      for (int e = 0; e < 16; ++e) tmax = fmaxf(tmax, sacc[e]);
      tmax = wave_max_xor32(tmax);
      const float m_new = fmaxf(m_run, tmax * scale_log2);
      const float m_ref = (m_new > m_run + 8.0f) ? m_new : m_run;
      const float alpha = __builtin_amdgcn_exp2f(m_run - m_ref);
      l_run *= alpha;
#pragma unroll
      for (int db = 0; db < DB; ++db) oacc[db] *= alpha;
      m_run = m_ref;
      settled = __builtin_amdgcn_readfirstlane(!careful && !__any(m_run == kUnseen));
    }
    // Weights 2^x, x = s * scale - m_run (log2 units), and O^T += V_tile^T P^T
    // in one run of code: the second half's exponentials run beside the first
    // half's MFMAs.  The normaliser sums the fp32 weights, before the bf16
    // rounding of the ones that enter P V, so that it and the LSE carry no bf16
    // error.
    float x[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) x[e] = __builtin_fmaf(sacc[e], scale_log2, -m_run);
    f32x8 pf[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
      for (int e = 0; e < 8; ++e) pf[ks][e] = __builtin_amdgcn_exp2f(x[8 * ks + e]);
      const bf16x8 pb = __builtin_convertvector(pf[ks], bf16x8);
#pragma unroll
      for (int db = 0; db < DB; ++db)
        oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vfrag[db][ks], pb, oacc[db], 0, 0, 0);
    }
    float s4[4];  // a tree of fp32 adds (short dependency chains)
#pragma unroll
    for (int i = 0; i < 4; ++i) s4[i] = (pf[0][i] + pf[0][i + 4]) + (pf[1][i] + pf[1][i + 4]);
    const float tsum = (s4[0] + s4[1]) + (s4[2] + s4[3]);
    l_run += tsum;
    // Weights above 256 (a sum <= 256 on every lane rules them out) went into O
    // and l as they are, in fp32 range; the reference moves up by a power of two
    // now, for the tiles to come.  A row's largest weights so far are among
    // them, so what their bf16 rounding left is added (V read from the stage
    // again: this is rare): with the reference moved to the tile's maximum
    // first, that one key's weight would be 1 and have no rounding error, and
    // without this the outputs' error against 64 bits is 0.9% larger (75k DiT
    // layer, 5 heads: 2.366e-3 against 2.344e-3).  A weight past fp32 range
    // leaves l or O infinite, which the end of the walk sees.  A careful walk
    // has moved its references already (lim is infinite).  A row that is NaN does
    // not count: for the other rows a residual of 0 or less times an infinite V
    // is NaN where the weights' product is infinite.
    if (__any(tsum > lim)) {
      moved = 1;
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        // Opaque, so that neither the rounded weights nor the V^T operands of
        // the product above are kept in registers for this (9 spilled).
#pragma unroll
        for (int e = 0; e < 8; ++e) asm volatile("" : "+v"(pf[ks][e]));
        const f32x8 pr = pf[ks] - __builtin_convertvector(__builtin_convertvector(pf[ks], bf16x8), f32x8);
        const bf16x8 pb = __builtin_convertvector(pr, bf16x8);
#pragma unroll
        for (int db = 0; db < DB; ++db) {
          uint32_t o0 = voff[db][0], o1 = voff[db][1];
          asm volatile("" : "+v"(o0), "+v"(o1));
          oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vread(ks, o0, o1), pb, oacc[db], 0, 0, 0);
        }
      }
      const float top = wave_max_xor32(tsum);
      const int up = top > 256.0f ? __builtin_amdgcn_frexp_expf(top) : 0;
      const float alpha = __builtin_amdgcn_ldexpf(1.0f, -up);
      l_run *= alpha;
#pragma unroll
      for (int db = 0; db < DB; ++db) oacc[db] *= alpha;
      m_run += static_cast<float>(up);
    }
  };
  // The walk, at most twice: a score more than ~119 (log2 units) above its
  // row's reference overflows a weight, which a test of every weight before
  // P V would catch in time (as the first tile does) at the price of the
  // softmax running beside no MFMA.  So O and l of a wave that met weights above
  // 256 (the others' are what a second walk would find) are tested once, at the
  // end: anything not finite sends the whole workgroup through the list again
  // with the references fixed before the weights.  Such a list costs
  // twice: 24 heads, 24001 tokens, a fifth of the keys, one key of every list
  // 200 nats above the others: 1.56 -> 3.26 ms (causal 0.81 -> 1.60, three
  // quarters of the blocks), where a test before each P V took 1.64 (0.88) and
  // 1.66 (0.90) on lists without such a key.
  for (;;) {
    if (ntiles > 0) {
#pragma unroll
      for (int n = 0; n < 2 * U; ++n) gather(n, 0);
      stage_ids(0, 0);
      load_ids(1);
    }
    int t = 0;
    for (; t + 2 < ntiles; t += 2) {
      step(t, 0, std::true_type{});
      step(t + 1, 1, std::true_type{});
    }
    if (t + 1 < ntiles) {
      step(t, 0, std::true_type{});
      step(t + 1, 1, std::false_type{});
    } else if (t < ntiles) {
      step(t, 0, std::false_type{});
    }
    if (moved && !careful) {
      float fin = l_run * 0.0f;  // 0, or NaN once anything is not finite
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int e = 0; e < 16; ++e) fin = __builtin_fmaf(oacc[db][e], 0.0f, fin);
      if (__any(fin != 0.0f) && lane == 0) s_redo = 1;
    }
    wait_vmcnt<0>();  // no gather may still be landing in the buffers the merge reuses
    __syncthreads();
    if (careful || !__builtin_amdgcn_readfirstlane(s_redo)) break;
    careful = 1;
    lim = INFINITY;
    settled = 0;
    m_run = kUnseen;
    l_run = 0.0f;
#pragma unroll
    for (int db = 0; db < DB; ++db) oacc[db] = f32x16{};
    if (ntiles > 0) load_ids(0);
  }

  if (herd && wave == 0 && lane == 0 && ntiles % kHerdBatch != 0)
    __hip_atomic_fetch_add(&g_herd[xcd * kHerdStride], kHerdUnit - herd_units(ntiles - ntiles % kHerdBatch),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);

  // Merge the two key halves (kw = 1 hands its state to kw = 0 through LDS).
  l_run += __shfl_xor(l_run, 32);
  // Reuse the tile buffers (each holds one row group's 32 x D fp32 O).
  float* red_o = reinterpret_cast<float*>(rw == 0 ? k_s0 : rw == 1 ? v_s0 : rw == 2 ? k_s1 : v_s1);
  float* red_ml = s_ml[rw];
  if (kw == 1) {
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int e = 0; e < 16; ++e) red_o[(db * 16 + e) * 64 + lane] = oacc[db][e];
    red_ml[lane] = m_run;
    red_ml[64 + lane] = l_run;
  }
  __syncthreads();
  if (kw == 1) return;

  const float m1 = red_ml[lane];
  const float l1 = red_ml[64 + lane];
  const float m = fmaxf(m_run, m1);
  float a0 = 0.0f, a1 = 0.0f, inv = 0.0f, l = 0.0f;
  if (m != kUnseen) {
    a0 = __builtin_amdgcn_exp2f(m_run - m);
    a1 = __builtin_amdgcn_exp2f(m1 - m);
    l = a0 * l_run + a1 * l1;
    inv = l > 0.0f ? 1.0f / l : 0.0f;
  }
  if (my_row >= row_end) return;
  if (lse && g == 0)
    lse[bh * N + my_row] = l > 0.0f ? (m + __builtin_log2f(l)) * 0.69314718055994531f : kNegInf;
  uint16_t* orow = o + b * o_sB + h * o_sH + static_cast<int64_t>(my_row) * o_sN;
#pragma unroll
  for (int db = 0; db < DB; ++db) {
#pragma unroll
    for (int vq = 0; vq < 4; ++vq) {
      f32x4 r;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int ee = 4 * vq + e;
        r[e] = (a0 * oacc[db][ee] + a1 * red_o[(db * 16 + ee) * 64 + lane]) * inv;
      }
      *reinterpret_cast<bf16x4*>(orow + 32 * db + 8 * vq + 4 * g) = __builtin_convertvector(r, bf16x4);
    }
  }
}

}  // namespace

// XCDs per group in the work mapping (1, 2, 4 or 8): the smallest group for
// which the K/V rows of the heads swept at once stay within ~160 MB, well inside
// the 256 MB last-level cache (the rest holds the Q, O and list streams).  One
// KV head's rows are N * D * 4 bytes (K and V, bf16), half of that under
// causal masking (a block's list spans the keys up to its own rows); the 8 / G
// groups sweep at most B * Hkv distinct KV heads.  Measured (attention alone):
// 75k-token DiT, 38.7 MB per head: 22.8 / 22.1 / 22.2 / 22.8 ms at G = 1 / 2 /
// 4 / 8; 119k-token DiT, 60.8 MB: 140.4 / 136.7 / 125 / 127 ms; causal VLM
// prefill at 131k tokens: G = 1 best by ~2%.
static int32_t xcd_group(int64_t N, int64_t D, int64_t Hkv, int64_t B, int32_t causal) {
  const double head_bytes = static_cast<double>(N) * static_cast<double>(D) * 4.0 *
                            (causal ? 0.5 : 1.0);
  const double budget = 160.0 * 1024.0 * 1024.0;
  for (int32_t g = 1; g < 8; g *= 2) {
    const double swept = static_cast<double>(std::min<int64_t>(8 / g, B * Hkv)) * head_bytes;
    if (swept <= budget) return g;
  }
  return 8;
}

// Workgroups of one sequence: group 0's share (the longest: its whole heads and
// its part of the heads left over; each of its XCDs takes every xgroup-th block
// of it), for all eight XCDs.
static int64_t sequence_grid(int64_t nheads, int32_t Np, int32_t chunks, int32_t xgroup) {
  const int64_t ngroups = 8 / xgroup, whole = nheads / ngroups;
  const int64_t seq0 = whole * Np + (nheads - whole * ngroups) * ((Np + ngroups - 1) / ngroups);
  return (seq0 + xgroup - 1) / xgroup * chunks * 8;
}

template <typename SEQS>
static hipError_t launch_grid(const SparseAttnArgs& a, int64_t grid, int32_t xgroup,
                              const SEQS& seqs, hipStream_t stream) {
  const int64_t B = a.q.B, Hq = a.q.H, N = a.q.N, D = a.q.D;
  const int32_t P = a.block;
  const int32_t Np = static_cast<int32_t>((N + P - 1) / P);
  const int32_t rows = P % 128 == 0 ? 128 : 64;
  const int32_t chunks = (P + rows - 1) / rows;
  const int64_t total = B * Hq * Np * chunks;
  const float scale = a.scale != 0.0f ? a.scale : 1.0f / sqrtf(static_cast<float>(D));
  const float scale_log2 = scale * 1.4426950408889634f;
  const int32_t group = static_cast<int32_t>(Hq / a.k.H);
  const uint16_t* q = static_cast<const uint16_t*>(a.q.ptr);
  const uint16_t* k = static_cast<const uint16_t*>(a.k.ptr);
  const uint16_t* v = static_cast<const uint16_t*>(a.v.ptr);
  uint16_t* o = static_cast<uint16_t*>(a.o);
  const bool same = a.k.sN == a.v.sN;
  auto launch = [&](auto kernel) -> hipError_t {
    // Workgroup slots per XCD (resident workgroups per CU x CUs per XCD).
    int dev = 0, cus = 0, per_cu = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    const int threads = 4 * rows;
    if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0);
    if (e != hipSuccess) return e;
    const int32_t slots = max(1, per_cu * cus / 8);
    hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(grid)), dim3(threads), 0, stream, q, a.q.sB,
                       a.q.sH, a.q.sN, k, a.k.sB, a.k.sH, a.k.sN, v, a.v.sB, a.v.sH, a.v.sN, o,
                       a.o_sB, a.o_sH, a.o_sN, a.lse, a.idx, a.counts, a.order, a.cap,
                       static_cast<int32_t>(Hq), group, static_cast<int32_t>(N), P, Np, chunks,
                       a.causal, scale_log2, total, xgroup, slots, seqs);
    return hipGetLastError();
  };
  if (rows == 128) {
    if (D == 128)
      return same ? launch(k_sparse_attn<128, true, 128, SEQS>) : launch(k_sparse_attn<128, false, 128, SEQS>);
    return same ? launch(k_sparse_attn<64, true, 128, SEQS>) : launch(k_sparse_attn<64, false, 128, SEQS>);
  }
  if (D == 128)
    return same ? launch(k_sparse_attn<128, true, 64, SEQS>) : launch(k_sparse_attn<128, false, 64, SEQS>);
  return same ? launch(k_sparse_attn<64, true, 64, SEQS>) : launch(k_sparse_attn<64, false, 64, SEQS>);
}

hipError_t launch_sparse_attn(const SparseAttnArgs& a, hipStream_t stream) {
  const int32_t P = a.block;
  const int32_t Np = static_cast<int32_t>((a.q.N + P - 1) / P);
  // 128 rows per workgroup when blocks come in multiples of 128 rows (one
  // gather of a tile then serves the whole block), else 64.
  const int32_t rows = P % 128 == 0 ? 128 : 64;
  const int32_t chunks = (P + rows - 1) / rows;
  const int64_t nheads = a.q.B * a.q.H;
  if (nheads * Np == 0) return hipSuccess;
  const int32_t xgroup = xcd_group(a.k.N, a.k.D, a.k.H, a.q.B, a.causal);
  return launch_grid(a, sequence_grid(nheads, Np, chunks, xgroup), xgroup, OneSeq{}, stream);
}

// A packed batch in one launch per kMaxSeqs sequences, longest first: launched
// one sequence at a time (longest blocks last), every sequence ended on a few
// workgroups and left the chip idle meanwhile.  Attention alone, 16 heads, causal
// / not: 30 sequences of 900 tokens 300 -> 143 / 372 -> 328 us, 20000 + 30000 +
// 5000 + 700 tokens 1158 -> 1016 / 2062 -> 1990, four of 16000 917 -> 871 / 1809
// -> 1680.
hipError_t launch_sparse_attn_varlen(const SparseAttnArgs& a, const int64_t* cu, int32_t nseq,
                                     hipStream_t stream) {
  const int32_t P = a.block;
  const int32_t rows = P % 128 == 0 ? 128 : 64;
  const int32_t chunks = (P + rows - 1) / rows;
  struct Seq {
    int64_t row0, len, first, grid;
    int32_t xgroup;
  };
  // Workgroups of one launch of several sequences (the grid's limit is 2^32
  // threads; a sequence on its own is launched whatever its size).
  constexpr int64_t kMaxGrid = int64_t(1) << 22;
  int64_t blocks = 0;
  for (int32_t s = 0; s < nseq;) {
    Seq seqs[kMaxSeqs];
    int32_t n = 0;
    int64_t grid = 0;
    for (; s < nseq && n < kMaxSeqs; ++s) {
      const int64_t len = cu[s + 1] - cu[s];
      if (len == 0) continue;
      const int32_t xgroup = xcd_group(len, a.k.D, a.k.H, 1, a.causal);
      const int64_t Np = (len + P - 1) / P;
      const int64_t g = sequence_grid(a.q.H, static_cast<int32_t>(Np), chunks, xgroup);
      if (n > 0 && grid + g > kMaxGrid) break;
      seqs[n++] = Seq{cu[s], len, blocks, g, xgroup};
      grid += g;
      blocks += Np;
    }
    if (n == 0) break;
    std::sort(seqs, seqs + n, [](const Seq& x, const Seq& y) {
      return x.len != y.len ? x.len > y.len : x.row0 < y.row0;
    });
    SeqTable t{};
    t.n = n;
    int64_t end = 0;
    for (int32_t x = 0; x < n; ++x) {
      end += seqs[x].grid;
      t.end[x] = static_cast<int32_t>(std::min<int64_t>(end, INT32_MAX));
      t.row0[x] = static_cast<int32_t>(seqs[x].row0);
      t.len[x] = static_cast<int32_t>(seqs[x].len);
      t.first[x] = static_cast<int32_t>(seqs[x].first);
      t.xgroup[x] = seqs[x].xgroup;
    }
    const hipError_t e = launch_grid(a, grid, t.xgroup[0], t, stream);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace vecattn
