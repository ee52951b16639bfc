// bf16 prompt phase on the gfx950 matrix cores.
//
//  attn_fwd   masked attention rows (Section 1; Section 3.1 Eq.3 of the paper): for a block
//             of query rows, K/V tiles of 64 keys stream through LDS, S^T = K Q^T and
//             O^T = V^T P^T run on v_mfma_f32_32x32x16_bf16 with an online softmax.
//             Writes O (optional) and the base-2 log-sum-exp of every row.
//  col_scores forgotten accumulated score of every key (Section 3.3 Eq.5):
//             S_j = sum_{i>=j} alpha^(n-1-i) * P[i, j].  A block of key columns stays in
//             registers, Q tiles stream through LDS, the logit tile is recomputed on the
//             matrix cores, exp2(s - lse_i + (n-1-i) log2 alpha) is formed per element (the
//             forgetting weight is folded into the exponent) and summed down the tile's
//             rows.  The n x n probability matrix is never written.
//  scores_select  column scores, selection and row moves of a short prompt or chunk in one kernel.
//
// All compute the TRANSPOSED logit tile (keys = M, queries = N).  In the 32x32
// accumulator layout a lane then owns one query (column l%32) and 16 keys
// (rows 8*(i/4) + 4*(l/32) + i%4, i = 0..15), so
//   - row statistics of the softmax are per-lane scalars (one exchange with lane^32),
//   - P^T is already in the B-operand layout of the second product (no LDS round trip),
//   - the column sums of col_scores accumulate per lane and are reduced across lanes once.
#include <math.h>

#include "a2sf_dev.h"
#include "a2sf_internal.h"
#include "select_dev.h"

namespace a2sf {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

constexpr int kTile = 64;  // keys (attn_fwd) or query rows (col_scores) per LDS tile
constexpr int kPrefetch = 4;  // LDS fragment reads in flight ahead of their matrix op

__device__ __forceinline__ f32x16 mfma_bf16(const uint4& a, const uint4& b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                 __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
// Older tokens in front of head gk's own keys; negative: the head is to be skipped.
__device__ __forceinline__ int rect_off(const AttnRect& rc, int gk) {
  if (!rc.off_heads) return 0;
  const int off = rc.off_heads[gk];
  return off <= rc.kv_stride - rc.m ? off : -1;
}
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Workgroup id -> flat work id such that each of the 8 accelerator dies (which receive
// consecutive workgroup ids round-robin) works on a contiguous range of work ids, i.e. on
// whole heads whose K/V stay in that die's L2.
__device__ __forceinline__ long long xcd_contiguous_id(long long total) {
  const long long per = (total + 7) / 8;
  return (long long)(blockIdx.x % 8) * per + blockIdx.x / 8;
}
// The order of the (head, block) items: that of ordered_item, or, for launches of up to RESIDENT blocks, head
// after head.  kOneRound: launches that are resident at once, where nothing is left to be dealt out and
// ordered_item costs half a microsecond.  kOnePerUnit, kTwoPerUnit: up to one, two workgroups per compute unit (attention: 100
// heads x 130, 200 blocks, 8.3 us and 10.4 in the order of ordered_item, 40 x 1000, 320 blocks, 26 and 23; scores: 45 x 1400,
// alpha = 0.9, 42 and 46).  Nor is there an order in one block per head.
constexpr long long kOneRound = 1ll << 62, kOnePerUnit = 256, kTwoPerUnit = 512;
template <long long RESIDENT>
__device__ __forceinline__ bool launch_item(int G, int nb, int& head, int& rank) {
  const long long total = (long long)G * nb;
  if (total > RESIDENT && nb > 1) return ordered_item(G, nb, head, rank);
  const long long id = xcd_contiguous_id(total);
  head = (int)(id / nb);
  rank = (int)(id % nb);
  return id < total;
}
template <long long RESIDENT>
unsigned launch_grid(int G, int nb) {
  const long long total = (long long)G * nb;
  return total > RESIDENT && nb > 1 ? ordered_grid(G, nb) : (unsigned)((total + 7) / 8 * 8);
}

// ---------------------------------------------------------------------------------------
// Masked attention rows, d = 64 or 128, on two gfx950 features:
//  * K and V tiles go from global memory straight into LDS (global_load_lds, 16 bytes per
//    lane, a wave fills 1 KB = 4 (d = 64: 8) rows per instruction; lane l's data lands at base + 16 l,
//    so the swizzle is applied by choosing which global chunk each lane fetches).  No
//    staging registers, no LDS store instructions.
//  * V stays row-major [key][d] in LDS; the V^T operand of O^T = V^T P^T is read with
//    ds_read_b64_tr_b16, which transposes 4x4 blocks of 16-bit elements across the 16
//    lanes of a group: output lane i, element r  <-  source lane 4r + i/4, element i%4.
//    Source lane (r, q) therefore points at V[key_r][d0 + 4q ..+3] and output lane i
//    receives V[key_0..3][d0 + i]: exactly the 4 consecutive keys of one half operand.
typedef short v4i16_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) char lds_char;

__device__ __forceinline__ uint2 lds_read_tr16(const lds_char* p) {
  v4i16_t r = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (__attribute__((address_space(3))) v4i16_t*)p);
  return __builtin_bit_cast(uint2, r);
}
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 lds_read16(const lds_char* p) {
  const u32x4_t r = *reinterpret_cast<const __attribute__((address_space(3))) u32x4_t*>(p);
  return make_uint4(r.x, r.y, r.z, r.w);
}

typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void lds_write8(lds_char* p, const uint2& v) {
  const u32x2_t x = {v.x, v.y};
  *reinterpret_cast<__attribute__((address_space(3))) u32x2_t*>(p) = x;
}

template <int D> constexpr int kTileBytesOf = kTile * D * 2;  // one 64-row tile
constexpr int kTileBytes = kTileBytesOf<128>;

// Chunk swizzles (16-byte chunks of a row; the LDS has 64 four-byte banks, i.e. 16 chunks side by
// side: one row of d = 128, two of d = 64).  K and Q are read 16 rows x one chunk column per 16
// lanes: XOR with the row (d = 64: row pair) spreads them over all 16 places.  V is read by 32
// lanes as 4 rows x 4 chunk columns x 2 halves: XOR with 4 * (row % 4) (d = 64: 4 * (row / 2 % 2))
// sends the rows to disjoint groups of four places.  Both measure zero LDS bank conflicts
// (SQ_LDS_BANK_CONFLICT).
template <int D = 128>
__device__ __forceinline__ int k_swizzle(int row) { return D == 128 ? (row & 15) : ((row >> 1) & 7); }
template <int D = 128>
__device__ __forceinline__ int v_swizzle(int row) { return D == 128 ? (row & 3) << 2 : ((row >> 1) & 1) << 2; }

// Geometry of a tile fetch: a wave's load u fills the rows (4 u + wave) * kRowsPerLoad ..
template <int D> constexpr int kRowsPerLoad = 512 / D;
template <int D> constexpr int kLoadsPerWave = kTile / (4 * kRowsPerLoad<D>);

template <int D, bool V_LAYOUT>
__device__ __forceinline__ void tile_place(int u, int& lrow, int& chunk) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) % kWaves;
  lrow = (u * 4 + wave) * kRowsPerLoad<D> + lane / (D / 8);
  chunk = (lane % (D / 8)) ^ (V_LAYOUT ? v_swizzle<D>(lrow) : k_swizzle<D>(lrow));
}
template <int D, bool V_LAYOUT>
__device__ __forceinline__ void dma_tile(const bf16_t* __restrict__ Mg, int row0, int n, lds_char* tile) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) % kWaves;
  const bf16_t* base = Mg + (size_t)row0 * D;
  const int most = n - 1 - row0;  // rows past the end repeat the last one
#pragma unroll
  for (int u = 0; u < kLoadsPerWave<D>; ++u) {
    int lrow, c;
    tile_place<D, V_LAYOUT>(u, lrow, c);
    dma16(base, (uint32_t)(min(lrow, most) * D * 2 + c * 16), (uint32_t)(size_t)(tile + (u * 4 + wave) * 1024));
  }
}

// dma_tile for a tile that straddles two sources: rows below `off` are rows of A, rows from
// `off` on are rows 0 .. of B (n rows in all).
template <int D, bool V_LAYOUT>
__device__ __forceinline__ void dma_tile2(const bf16_t* __restrict__ A, const bf16_t* __restrict__ B,
                                          int off, int row0, int n, lds_char* tile) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) % kWaves;
#pragma unroll
  for (int u = 0; u < kLoadsPerWave<D>; ++u) {
    int lrow, c;
    tile_place<D, V_LAYOUT>(u, lrow, c);
    const int r = min(row0 + lrow, n - 1);
    const bf16_t* src = r < off ? A + (size_t)r * D : B + (size_t)(r - off) * D;
    dma16_at(src + c * 8, (uint32_t)(size_t)(tile + (u * 4 + wave) * 1024));
  }
}

// Same as dma_tile for a tile that lies completely inside the matrix: the per-lane byte
// offsets `loff` (row-in-tile and swizzled chunk) are loop invariants, the tile base is
// wave-uniform, so a tile costs its load instructions and no address arithmetic per lane.
template <int D, bool V_LAYOUT>
__device__ __forceinline__ void dma_offsets(int (&loff)[kLoadsPerWave<D>]) {
#pragma unroll
  for (int u = 0; u < kLoadsPerWave<D>; ++u) {
    int lrow, c;
    tile_place<D, V_LAYOUT>(u, lrow, c);
    loff[u] = lrow * D * 2 + c * 16;
  }
}
template <int D>
__device__ __forceinline__ void dma_full_tile(const bf16_t* __restrict__ Mg, int row0,
                                              const int (&loff)[kLoadsPerWave<D>], lds_char* tile) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) % kWaves;
  const bf16_t* base = Mg + (size_t)row0 * D;
#pragma unroll
  for (int u = 0; u < kLoadsPerWave<D>; ++u) dma16(base, (uint32_t)loff[u], (uint32_t)(size_t)(tile + (u * 4 + wave) * 1024));
}

// With outputs a wave works one tile ahead of itself: while the vector ALU forms the
// probabilities of tile t, the matrix pipe forms the logits of tile t + 1 (the two are
// interleaved in the instruction stream), then O += V(t)^T P(t).  K tiles are fetched two steps ahead,
// V tiles one.  Exponentials are taken against the running maximum as it is, without looking for
// the tile's own: floating point keeps their relative precision whatever their size, so the
// maximum has to move (and O to be rescaled) only when a tile's sum leaves a range (or is not a number: the
// first tile, whose running maximum is -inf).  Sums alone may grow to 2^30; with outputs a probability stays below
// 2^8, so that O overflows for values above 2^120 / (number of keys) only.
constexpr float kMoveMaximumAt = 1073741824.f, kMoveMaximumWithO = 256.f;

// KS = 2 (with outputs): eight waves, the second four take the odd tiles of the same 128 rows and the
// two halves are merged at the end -- for launches that do not fill the chip, where the chain of
// tiles of a head's last rows is what the call waits for.
// PIPED = false (with outputs): a tile's logits, probabilities and products one after the other, no work for a tile that
// is not there -- for rows of a few tiles, where the start of the pipeline is most of the time.
template <int D, bool WITH_O, int KS, bool PIPED>
__global__ __launch_bounds__(kThreads * KS, !WITH_O ? 4 : 2 / KS) void attn_fwd_kernel(
    const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, const bf16_t* __restrict__ V,
    bf16_t* __restrict__ O, float* __restrict__ LSE2, AttnRect rc, int G, int nqb, float scale_log2e) {
  constexpr int BM = kWaves * 32, KK = D / 16, DB = D / 32, ROW = D * 2;
  constexpr int kTB = kTileBytesOf<D>, NL = kLoadsPerWave<D>;
  // two stages of K tiles, two of V tiles (none without outputs; a deeper ring was measured for
  // that pass and is slower: it costs occupancy)
  // (with outputs: and 4 KB that take the loads of a step that has nothing to fetch)
  constexpr int kLds = !WITH_O ? 2 * kTB : 4 * kTB + (PIPED ? 4096 : 0);
  __shared__ __attribute__((aligned(1024))) char smem[KS * kLds];
  __shared__ float m_other[KS > 1 ? BM : 1], l_other[KS > 1 ? BM : 1];

  int g, rank;
  if (!launch_item<KS == 1 ? kOnePerUnit : kOneRound>(G, nqb, g, rank)) return;
  // the launch covers the nqb row blocks from the one that holds rc.first_row on
  const int qb = rc.first_row / BM + nqb - 1 - rank;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6) % kWaves;  // wave-uniform: branches on it are scalar
  const int part = KS > 1 ? __builtin_amdgcn_readfirstlane(tid >> 6) / kWaves : 0;  // of the tiles: part, part + KS, ...
  lds_char* const lds = (lds_char*)smem + part * kLds;
  const int l32 = lane & 31, h = lane >> 5;
  const int n = rc.m;
  const int gk = g / rc.kv_group;  // the K/V head this query head reads
  const int off = rect_off(rc, gk);
  const int row0 = qb * BM;
  if (off < 0) {  // a head the caller's precondition excludes: its rows are flagged with NaN
    if (WITH_O)
      for (int e = tid; e < min(BM, n - row0) * D; e += kThreads * KS)
        O[((size_t)g * n + row0) * D + e] = (bf16_t)0x7FC0;
    return;
  }
  const int nk = off + n;  // keys of this head
  const bf16_t* Qg = Q + (size_t)g * n * D;
  const bf16_t* Kg = K + (size_t)gk * rc.kv_stride * D;
  const bf16_t* Vg = V + (size_t)gk * rc.kv_stride * D;
  // second source (keys off .. off+n-1), or null
  const bf16_t* K2g = rc.k2 ? (const bf16_t*)rc.k2 + (size_t)gk * n * D : nullptr;
  const bf16_t* V2g = rc.k2 ? (const bf16_t*)rc.v2 + (size_t)gk * n * D : nullptr;
  const int wrow0 = row0 + wave * 32;  // first query row of this wave

  // Q fragments (B operand): lane (query l32, half h) holds Q[query][16kk + 8h .. +7]
  uint4 qf[KK];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) qf[kk] = load16(Qg + (size_t)min(wrow0 + l32, n - 1) * D + kk * 16 + h * 8);
  // per-lane LDS byte offsets inside a K / V tile
  int koff[KK];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) koff[kk] = l32 * ROW + (((2 * kk + h) ^ k_swizzle<D>(l32)) << 4);
  int voff[DB];
  {
    const int i = lane & 15, r = i >> 2, qd = i & 3, gq = (lane >> 4) & 1;
    const int cl = 2 * gq + (qd >> 1), vs = v_swizzle<D>(4 * h + r);  // key = 8*x + 4h + r
#pragma unroll
    for (int db = 0; db < DB; ++db) voff[db] = (4 * h + r) * ROW + ((((4 * db + cl) ^ vs)) << 4) + (qd & 1) * 8;
  }

  const int last_key = off + min(n, row0 + BM) - 1;  // newest key the block's rows see
  const int ntiles = last_key / kTile + 1;
  int k_loff[NL], v_loff[NL];
  dma_offsets<D, false>(k_loff);
  if (WITH_O) dma_offsets<D, true>(v_loff);
  auto fetch_k = [&](int t, lds_char* buf) {
    if (K2g && (t + 1) * kTile > off) {       // the tile holds rows of the second source
      if (t * kTile >= off && (t + 1) * kTile <= nk) dma_full_tile<D>(K2g, t * kTile - off, k_loff, buf);
      else dma_tile2<D, false>(Kg, K2g, off, t * kTile, nk, buf);
    } else if ((t + 1) * kTile <= nk) {
      dma_full_tile<D>(Kg, t * kTile, k_loff, buf);
    } else {
      dma_tile<D, false>(Kg, t * kTile, nk, buf);
    }
  };
  auto fetch_v = [&](int t, lds_char* buf) {
    if (K2g && (t + 1) * kTile > off) {
      if (t * kTile >= off && (t + 1) * kTile <= nk) dma_full_tile<D>(V2g, t * kTile - off, v_loff, buf);
      else dma_tile2<D, true>(Vg, V2g, off, t * kTile, nk, buf);
    } else if ((t + 1) * kTile <= nk) {
      dma_full_tile<D>(Vg, t * kTile, v_loff, buf);
    } else {
      dma_tile<D, true>(Vg, t * kTile, nk, buf);
    }
  };
  lds_char* const vst = lds + 2 * kTB;  // the V stages
  if (part < ntiles) fetch_k(part, lds);
  if (WITH_O) {
    if (part < ntiles) fetch_v(part, vst);
    if (PIPED && part + KS < ntiles) fetch_k(part + KS, lds + kTB);
  }
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) asm volatile("" : "+v"(qf[kk].x));  // waited for here, not in the loop
  wait_vm_barrier<0>();

  float m = -INFINITY, lsum = 0.f;
  const int newest = off + wrow0 + l32;  // newest key this lane's row sees
  const int nt_wave = min(ntiles, (off + wrow0 + 31) / kTile + 1);  // tiles with a key this wave's rows see
  // steps of the workgroup, and those with a tile for this wave (step u: tile part + KS u)
  const int steps = (ntiles + KS - 1) / KS, steps_wave = nt_wave > part ? (nt_wave - part + KS - 1) / KS : 0;
  // the 32 logits of a lane (its query against the keys 32 kb + 8 (i/4) + 4h + i%4 of tile t)
  auto logits = [&](const lds_char* kt, f32x16 (&s)[2], auto between) {
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int i = 0; i < 16; ++i) s[kb][i] = 0.f;
    constexpr int NF = 2 * KK;  // fragment i = (kk, kb): the two key blocks alternate, so that no
    uint4 fr[NF];               // matrix op waits for the one before it
#pragma unroll
    for (int i = 0; i < kPrefetch; ++i) fr[i] = lds_read16(kt + (i & 1) * 32 * ROW + koff[i >> 1]);
#pragma unroll
    for (int i = 0; i < NF; ++i) {
      if (i + kPrefetch < NF) fr[i + kPrefetch] = lds_read16(kt + ((i + kPrefetch) & 1) * 32 * ROW + koff[(i + kPrefetch) >> 1]);
      s[i & 1] = mfma_bf16(fr[i], qf[i >> 1], s[i & 1]);
      between(i);
    }
  };
  auto mask = [&](int t, f32x16 (&s)[2]) {  // causal, where tile t reaches past the wave's first row
    if (t * kTile + kTile - 1 > off + wrow0) {
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (t * kTile + kb * 32 + 8 * (i >> 2) + 4 * h + (i & 3) > newest) s[kb][i] = -INFINITY;
    }
  };
  // a new running maximum that covers the tile (rare); returns the factor older sums shrink by
  auto move_maximum = [&](const f32x16 (&s)[2]) {
    float mx = s[0][0];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int i = 0; i < 16; ++i) mx = fmaxf(mx, s[kb][i]);
    mx = across_rows(mx, OpMax(), false, true);
    // (rows past the end of a ragged block can be fully masked: keep m finite)
    const float m_new = fmaxf(m, fmaxf(mx * scale_log2e, -1e30f));
    const float corr = fast_exp2(m - m_new);  // 0 on the first tile
    m = m_new;
    return corr;
  };

  const auto keep_reads_ahead = [] {  // in `logits`: kPrefetch reads up front, then one new read per matrix op
    __builtin_amdgcn_sched_group_barrier(0x100, kPrefetch, 0);
#pragma unroll
    for (int i = 0; i < 2 * KK; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      if (i + kPrefetch < 2 * KK) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
  };

  if constexpr (!WITH_O) {
    auto tile_step = [&](int t, const lds_char* kt) {
      if (t >= nt_wave) return;
      f32x16 s[2];
      logits(kt, s, [](int) {});
      keep_reads_ahead();
      mask(t, s);
      float rs = 0.f;
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int i = 0; i < 16; ++i) rs += fast_exp2(fmaf(s[kb][i], scale_log2e, -m));
      if (__any(!(rs < kMoveMaximumAt))) {
        lsum *= move_maximum(s);
        rs = 0.f;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
          for (int i = 0; i < 16; ++i) rs += fast_exp2(fmaf(s[kb][i], scale_log2e, -m));
      }
      lsum += rs;
    };
    for (int t0 = 0; t0 < ntiles; t0 += 2) {
#pragma unroll
      for (int b = 0; b < 2; ++b) {  // stage t % 2: LDS offsets are immediates
        const int t = t0 + b;
        if (t >= ntiles) break;
        // the stage of tile t - 1 is free: every wave passed the barrier that ended its step
        if (t + 1 < ntiles) fetch_k(t + 1, lds + (1 - b) * kTB);
        tile_step(t, lds + b * kTB);
        wait_vm_barrier<0>();  // tile t + 1 for every wave of the workgroup
      }
    }
    const float l = across_rows(lsum, OpAdd(), false, true);
    if (wrow0 + l32 < n && h == 0) LSE2[(size_t)g * n + wrow0 + l32] = m + log2f(l);
  } else {
    f32x16 oacc[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int i = 0; i < 16; ++i) oacc[db][i] = 0.f;
    const auto add_values = [&](const lds_char* vt, const uint32_t (&pf)[16]) {  // O += V^T P
      constexpr int NF = DB * 4;  // fragment i = (kb, tt, db), db fastest
      uint2 lo[NF], hi[NF];
      auto vread = [&](int i, uint2& a, uint2& b) {
        const lds_char* p = vt + ((i / DB) * 16) * ROW + voff[i % DB];
        a = lds_read_tr16(p);
        b = lds_read_tr16(p + 8 * ROW);
      };
#pragma unroll
      for (int i = 0; i < kPrefetch; ++i) vread(i, lo[i], hi[i]);
#pragma unroll
      for (int i = 0; i < NF; ++i) {
        if (i + kPrefetch < NF) vread(i + kPrefetch, lo[i + kPrefetch], hi[i + kPrefetch]);
        const int w = 4 * (i / DB);
        oacc[i % DB] = mfma_bf16(make_uint4(lo[i].x, lo[i].y, hi[i].x, hi[i].y),
                                 make_uint4(pf[w], pf[w + 1], pf[w + 2], pf[w + 3]), oacc[i % DB]);
      }
      __builtin_amdgcn_sched_group_barrier(0x100, 2 * kPrefetch, 0);
#pragma unroll
      for (int i = 0; i < NF; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        if (i + kPrefetch < NF) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
      }
    };
    if constexpr (!PIPED) {
      for (int t0 = 0; t0 < ntiles; t0 += 2) {
#pragma unroll
        for (int b = 0; b < 2; ++b) {  // stage t % 2: LDS offsets are immediates
          const int t = t0 + b;
          if (t >= ntiles) break;
          // the stages of tile t - 1 are free: every wave passed the barrier that ended its step
          if (t + 1 < ntiles) {
            fetch_k(t + 1, lds + (1 - b) * kTB);
            fetch_v(t + 1, vst + (1 - b) * kTB);
          }
          if (t < nt_wave) {
            f32x16 s[2];
            logits(lds + b * kTB, s, [](int) {});
            keep_reads_ahead();
            mask(t, s);
            float mx = s[0][0];
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
              for (int i = 0; i < 16; ++i) mx = fmaxf(mx, s[kb][i]);
            mx = fmaxf(across_rows(mx, OpMax(), false, true) * scale_log2e, -1e30f);
            if (__any(mx > m + 8.f)) {  // (kMoveMaximumWithO is 2^8)
              const float m_new = fmaxf(m, mx), corr = fast_exp2(m - m_new);
              lsum *= corr;
#pragma unroll
              for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int i = 0; i < 16; ++i) oacc[db][i] *= corr;
              m = m_new;
            }
            uint32_t pf[16];
            float rs = 0.f;
#pragma unroll
            for (int j = 0; j < 16; ++j) {
              const float e0 = fast_exp2(fmaf(s[j >> 3][(2 * j) & 15], scale_log2e, -m));
              const float e1 = fast_exp2(fmaf(s[j >> 3][(2 * j + 1) & 15], scale_log2e, -m));
              rs += e0;
              rs += e1;
              pf[j] = pack_bf16(e0, e1);
            }
            lsum += rs;
            add_values(vst + b * kTB, pf);
          }
          wait_vm_barrier<0>();  // tile t + 1 for every wave of the workgroup
        }
      }
    } else {
      f32x16 sa[2], sb[2];
      logits(lds, sa, [](int) {});
      // every wave is done with K(0) before K(2) takes its place
      wait_vm_barrier<0>();

      // probabilities of tile t (logits in s) beside the logits of tile t + 1 (into s_next; past the
      // wave's last tile they are formed from whatever the stage holds and not used), then O += V^T P
      //
      // The loads of a tile are issued one by one between the first matrix ops: a load of 1 KB keeps
      // the compute unit's one address path busy for 16 cycles, and issued at once after the barrier the
      // eight loads of all waves held every wave up for 700 of the 2800 cycles of a step.  So that the
      // instruction stream is the same in every step, a step without a whole tile to fetch (none left;
      // or a ragged or two-source tile, which was fetched before) sends its loads to the spare 4 KB.
      // (all lanes then read the head's first 16 bytes of Q, which every head has.)
      struct Fetch {
        const char* from;
        uint32_t to, stride, lanes;  // lanes: mask of the per-lane offsets
      };
      const uint32_t spare = (uint32_t)(size_t)(lds + 4 * kTB) + wave * 1024;
      const auto whole_k = [&](int t, lds_char* buf) -> Fetch {
        const uint32_t to = (uint32_t)(size_t)buf + wave * 1024;
        if (t < ntiles) {
          if (K2g && (t + 1) * kTile > off) {
            if (t * kTile >= off && (t + 1) * kTile <= nk)
              return {reinterpret_cast<const char*>(K2g + (size_t)(t * kTile - off) * D), to, 4096u, ~0u};
            dma_tile2<D, false>(Kg, K2g, off, t * kTile, nk, buf);
          } else if ((t + 1) * kTile <= nk) {
            return {reinterpret_cast<const char*>(Kg + (size_t)t * kTile * D), to, 4096u, ~0u};
          } else {
            dma_tile<D, false>(Kg, t * kTile, nk, buf);
          }
        }
        return {reinterpret_cast<const char*>(Qg), spare, 0u, 0u};
      };
      const auto whole_v = [&](int t, lds_char* buf) -> Fetch {
        const uint32_t to = (uint32_t)(size_t)buf + wave * 1024;
        if (t < ntiles) {
          if (K2g && (t + 1) * kTile > off) {
            if (t * kTile >= off && (t + 1) * kTile <= nk)
              return {reinterpret_cast<const char*>(V2g + (size_t)(t * kTile - off) * D), to, 4096u, ~0u};
            dma_tile2<D, true>(Vg, V2g, off, t * kTile, nk, buf);
          } else if ((t + 1) * kTile <= nk) {
            return {reinterpret_cast<const char*>(Vg + (size_t)t * kTile * D), to, 4096u, ~0u};
          } else {
            dma_tile<D, true>(Vg, t * kTile, nk, buf);
          }
        }
        return {reinterpret_cast<const char*>(Qg), spare, 0u, 0u};
      };
      auto tile_step = [&](int t, const lds_char* kt_next, const lds_char* vt, f32x16 (&s)[2], f32x16 (&s_next)[2],
                           const Fetch& fk, const Fetch& fv) {
        const auto piece = [&](int i) {
          if (i < NL) dma16(fk.from, (uint32_t)k_loff[i] & fk.lanes, fk.to + i * fk.stride);
          else if (i < 2 * NL) dma16(fv.from, (uint32_t)v_loff[i - NL] & fv.lanes, fv.to + (i - NL) * fv.stride);
        };
        mask(t, s);
        float rs = 0.f, e0 = 0.f, e1 = 0.f;
        uint32_t pf[16];  // bf16 probabilities 2j, 2j + 1 (of the lane's 32, key block by key block)
        const auto finish = [&](int j) {  // the pair whose exponentials were requested last
          rs += e0;
          rs += e1;
          pf[j] = pack_bf16(e0, e1);
        };
        // between two matrix ops: a load, and the lane's share of the probabilities -- no result is used
        // right behind the instruction that forms it
        logits(kt_next, s_next, [&](int i) {
          if (i < 2 * NL) piece(i);
          constexpr int PAIRS = 16 / (2 * KK);
#pragma unroll
          for (int jj = 0; jj < PAIRS; ++jj) {
            const int j = PAIRS * i + jj;
            const float x0 = fmaf(s[j >> 3][(2 * j) & 15], scale_log2e, -m), x1 = fmaf(s[j >> 3][(2 * j + 1) & 15], scale_log2e, -m);
            if (j > 0) finish(j - 1);
            e0 = fast_exp2(x0);
            e1 = fast_exp2(x1);
          }
          __builtin_amdgcn_sched_barrier(0);
        });
        finish(15);
        if (__any(!(rs < kMoveMaximumWithO))) {
          const float corr = move_maximum(s);
          lsum *= corr;
#pragma unroll
          for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int i = 0; i < 16; ++i) oacc[db][i] *= corr;
          rs = 0.f;
#pragma unroll
          for (int j = 0; j < 16; ++j) {
            e0 = fast_exp2(fmaf(s[j >> 3][(2 * j) & 15], scale_log2e, -m));
            e1 = fast_exp2(fmaf(s[j >> 3][(2 * j + 1) & 15], scale_log2e, -m));
            finish(j);
          }
        }
        lsum += rs;
        add_values(vt, pf);
      };

      for (int u0 = 0; u0 < steps_wave; u0 += 2) {
#pragma unroll
        for (int b = 0; b < 2; ++b) {  // stage u % 2: LDS offsets are immediates
          if (u0 + b >= steps_wave) break;
          const int t = part + KS * (u0 + b);
          // free since the last barrier: the stages of K(u), whose logits are formed, and of V(u-1)
          const Fetch fk = whole_k(t + 2 * KS, lds + b * kTB), fv = whole_v(t + KS, vst + (1 - b) * kTB);
          if (b == 0) tile_step(t, lds + kTB, vst, sa, sb, fk, fv);
          else tile_step(t, lds, vst + kTB, sb, sa, fk, fv);
          wait_vm_barrier<0>();  // K(u+2) and V(u+1) for every wave of the workgroup
        }
      }
      // tiles that only the workgroup's later rows see: the wave still fetches its quarter
      for (int u = steps_wave; u < steps; ++u) {
        const int t = part + KS * u;
        if (t + 2 * KS < ntiles) fetch_k(t + 2 * KS, lds + (u & 1) * kTB);
        if (t + KS < ntiles) fetch_v(t + KS, vst + (1 - (u & 1)) * kTB);
        wait_vm_barrier<0>();
      }
    }
    // ---- epilogue.  The accumulator layout gives a lane 4 consecutive d of one row at a time:
    // written straight to memory that is 32 rows x 16 bytes per instruction.  Instead each wave
    // transposes its 32 x D output block through its own strip of LDS (free after the
    // loop's last barrier; 16-byte chunks XOR-swizzled by the row) and stores whole rows, 1 KB per
    // instruction.
    float l = across_rows(lsum, OpAdd(), false, true);
    if constexpr (KS > 1) {
      // the second half's sums, through the rings (free after the loop's last barrier)
      typedef __attribute__((address_space(3))) f32x4_t lds_f32x4;
      static_assert(kWaves * DB * 4 * 1024 <= KS * kLds, "a register quad of all lanes per KB");
      lds_char* const osum = (lds_char*)smem + wave * (DB * 4 * 1024) + lane * 16;
      if (part == 1) {
        if (h == 0) { m_other[wave * 32 + l32] = m; l_other[wave * 32 + l32] = l; }
#pragma unroll
        for (int i = 0; i < 4 * DB; ++i)
          *reinterpret_cast<lds_f32x4*>(osum + i * 1024) =
              f32x4_t{oacc[i >> 2][4 * (i & 3)], oacc[i >> 2][4 * (i & 3) + 1], oacc[i >> 2][4 * (i & 3) + 2], oacc[i >> 2][4 * (i & 3) + 3]};
      }
      __syncthreads();
      if (part == 1) return;
      const float m1 = m_other[wave * 32 + l32], l1 = l_other[wave * 32 + l32];
      const float m_all = fmaxf(m, m1);  // this half has seen key 0: finite
      const float f0 = fast_exp2(m - m_all), f1 = fast_exp2(m1 - m_all);  // 0 for a half without tiles
      l = l * f0 + l1 * f1;
      m = m_all;
#pragma unroll
      for (int i = 0; i < 4 * DB; ++i) {
        const f32x4_t x = *reinterpret_cast<const lds_f32x4*>(osum + i * 1024);
#pragma unroll
        for (int e = 0; e < 4; ++e) oacc[i >> 2][4 * (i & 3) + e] = oacc[i >> 2][4 * (i & 3) + e] * f0 + x[e] * f1;
      }
    }
    if (wrow0 + l32 < n && h == 0) LSE2[(size_t)g * n + wrow0 + l32] = m + log2f(l);
    // (with KS = 2 the merged waves' strips lie above what they read: the second ring)
    lds_char* const ostrip = (lds_char*)smem + (KS - 1) * kLds + wave * 32 * ROW;
    const float inv = 1.0f / l;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4) {
        uint2 w;
        w.x = pack_bf16(oacc[db][4 * i4 + 0] * inv, oacc[db][4 * i4 + 1] * inv);
        w.y = pack_bf16(oacc[db][4 * i4 + 2] * inv, oacc[db][4 * i4 + 3] * inv);
        // row l32, elements 32db + 8*i4 + 4h .. +3  ->  chunk 4db + i4, half h
        lds_write8(ostrip + l32 * ROW + (((4 * db + i4) ^ k_swizzle<D>(l32)) << 4) + 8 * h, w);
      }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    __builtin_amdgcn_wave_barrier();
    constexpr int RPL = kRowsPerLoad<D>;
    const int rr = lane / (D / 8), c = lane % (D / 8);
#pragma unroll
    for (int u = 0; u < 32 / RPL; ++u) {
      const int r = RPL * u + rr;
      const uint4 x = lds_read16(ostrip + r * ROW + ((c ^ k_swizzle<D>(r)) << 4));
      if (wrow0 + r < n) store16(O + ((size_t)g * n + wrow0 + r) * D + c * 8, x);
    }
  }
}

// ---------------------------------------------------------------------------------------
// d = 128 with two 32-row query blocks per wave (64 rows per wave, 256 per workgroup) and one
// wave per SIMD.  Same operand conventions, LDS tile layouts and mathematics as
// attn_fwd_kernel; the instruction stream (register map, phase schedule, hazards) is
// written by gen_attn_fwd128x2.py, whose header describes it.  This wrapper derives the
// per-lane offsets and per-wave pointers and hands them to that stream.  Requires
// n % 256 == 0 and an output pointer.
#include "attn_fwd128x2_body.inc"
#include "attn_fwd128x2r_body.inc"

constexpr int kX2Rows = 256;             // query rows per workgroup and block
constexpr int kX2RingBytes = 4 * 32768;  // four stages of one K tile + one V tile
constexpr int kX2LdsBytes = kX2RingBytes + 4 * 8192;  // + one 8 KB output strip per wave
constexpr int kX2MinRows = 512;
constexpr int kX2Slots = 32;             // persistent launch: workgroups per XCD (one per CU)

// rounds == 1: one workgroup per (head, 256-row block), ids mapped as in the other kernels.
// rounds > 1 (persistent launch, 8 * kX2Slots workgroups, nqb a power of two): the workgroup
// in slot r of XCD x works on ids x * (total / 8) + r + 32 j, j = 0 .. rounds - 1; the K/V tile
// stream runs on from one block into the next and a block's Q rows are loaded during the last
// tile of the block before, so a block starts with its first tiles already in LDS.
__global__ __launch_bounds__(kThreads, 1) void attn_fwd128x2_kernel(
    const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, const bf16_t* __restrict__ V,
    bf16_t* __restrict__ O, float* __restrict__ LSE2, int n, int nqb, int id_base, int ids,
    int rounds, int kv_shift, unsigned kv_magic, float scale_log2e) {
  // query head g reads the keys and values of K/V head g / r (grouped-query heads) =
  // mulhi(g, kv_magic) + (g >> kv_shift): r a power of two: kv_magic = 0, kv_shift = log2 r;
  // otherwise kv_shift = 31 and kv_magic = floor(2^32 / r) + 1
  __shared__ __attribute__((aligned(1024))) char smem[kX2LdsBytes];
  // this launch covers the ids id_base .. id_base + ids - 1; id = head * nqb + block position
  int vid0;
  if (rounds > 1) {
    vid0 = id_base + (int)(blockIdx.x % 8) * (ids / 8) + (int)(blockIdx.x / 8);
  } else {
    const long long vid = xcd_contiguous_id(ids);
    if (vid >= ids) return;
    vid0 = id_base + (int)vid;
  }
  const int g0 = vid0 / nqb;
  const int qb0 = nqb - 1 - vid0 % nqb;  // longest rows first
  const int lgnqb = 31 - __builtin_clz(nqb), nqbm1 = nqb - 1;  // used from the second round on

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l32 = lane & 31, h = lane >> 5;
  const unsigned lds0 = (unsigned)(size_t)smem;  // LDS byte address of the stage ring

  // K fragment (16 d-chunk 2kk+h of key row l32): row base and the kk-independent swizzle term
  const unsigned krow = lds0 + l32 * 256, hx16 = (unsigned)((h ^ k_swizzle(l32)) << 4);
  // V fragment (see attn_fwd_kernel): source lane (r, qd) of group gq, key rows 4h + r
  const int i16 = lane & 15, r4 = i16 >> 2, qd = i16 & 3, gq = (lane >> 4) & 1;
  const unsigned clvs16 = (unsigned)(((2 * gq + (qd >> 1)) ^ v_swizzle(r4)) << 4);
  const unsigned vrow = lds0 + kTileBytes + (4 * h + r4) * 256 + (qd & 1) * 8;
  // DMA: this wave fills rows 16u + 4 wave + rr of a tile, lane (rr, pc) the chunk slot pc
  const int rr = lane >> 4, pc = lane & 15, lrow = 4 * wave + rr;
  const unsigned kl0 = (unsigned)(lrow * 256 + ((pc ^ k_swizzle(lrow)) << 4));
  const unsigned vl0 = (unsigned)(lrow * 256 + ((pc ^ v_swizzle(lrow)) << 4));
  const unsigned qoff = (unsigned)(l32 * 256 + h * 16);
  const int lv = l32 - 4 * h;
  const unsigned l32x4 = l32 * 4, lanex16 = lane * 16;
  // epilogue: a wave's 32 x 128 output blocks go, one after the other, through its own 8 KB
  // strip of LDS above the ring
  const unsigned strip = lds0 + kX2RingBytes + wave * 8192;
  const unsigned strip_w = strip + l32 * 256 + 8 * h, x16 = (unsigned)((l32 & 15) << 4);
  const unsigned strip_r = strip + rr * 256, crr16 = (unsigned)((pc ^ rr) << 4);

  // Rows: a 256-row block is cut into eight 32-row blocks; wave w owns blocks w ("block 0")
  // and 7 - w ("block 1"), so that every wave has the same number of key tiles to go through
  // although the rows further down see more keys.
  const int w32a = 32 * wave, w32b = 32 * (7 - wave), wodd = wave & 1;
  const unsigned wave_lds = lds0 + wave * 1024;
  const unsigned long long qa = (unsigned long long)Q, ka = (unsigned long long)K,
                           va = (unsigned long long)V, oa = (unsigned long long)O,
                           la = (unsigned long long)LSE2;

  asm volatile(A2SF_FWD128X2_ASM
               :
               : [hx16] "v"(hx16), [krow] "v"(krow), [clvs16] "v"(clvs16), [vrow] "v"(vrow),
                 [kl0] "v"(kl0), [vl0] "v"(vl0), [qoff] "v"(qoff), [lv] "v"(lv),
                 [l32x4] "v"(l32x4), [lanex16] "v"(lanex16), [strip_w] "v"(strip_w),
                 [x16] "v"(x16), [crr16] "v"(crr16), [strip_r] "v"(strip_r),
                 [qlo] "s"((unsigned)qa), [qhi] "s"((unsigned)(qa >> 32)),
                 [klo] "s"((unsigned)ka), [khi] "s"((unsigned)(ka >> 32)),
                 [vlo] "s"((unsigned)va), [vhi] "s"((unsigned)(va >> 32)),
                 [olo] "s"((unsigned)oa), [ohi] "s"((unsigned)(oa >> 32)),
                 [llo] "s"((unsigned)la), [lhi] "s"((unsigned)(la >> 32)),
                 [n] "s"(n), [g0] "s"(g0), [qb0] "s"(qb0), [vid0] "s"(vid0), [rounds] "s"(rounds),
                 [lgnqb] "s"(lgnqb), [nqbm1] "s"(nqbm1), [w32a] "s"(w32a), [w32b] "s"(w32b),
                 [wodd] "s"(wodd), [wave_lds] "s"(wave_lds), [kvs] "s"(kv_shift), [kvm] "s"(kv_magic),
                 [scale] "s"(scale_log2e)
               : A2SF_FWD128X2_CLOBBERS);
}

// The same for any n >= 512 and any number of row blocks per head (nqb = ceil(n / 256)): the stream
// that clamps the fetches and narrows the stores of a head's last row block.
// rounds > 1 (8 * kX2Slots workgroups): the work is the pairs P = a * nqb + p, (row block
// nqb - 1 - p of head 2a, row block p of head 2a + 1); the workgroup in slot r of XCD x takes the
// pairs x * (pairs / 8) + r + 32 k, k = 0 .. rounds / 2 - 1.
// rounds == 1: first the `odd` blocks of a head without partner (head GQ - 1), longest first, then
// the longer blocks of the pairs pair_base .. pair_base + pairs - 1, then the shorter ones.
__global__ __launch_bounds__(kThreads, 1) void attn_fwd128x2r_kernel(
    const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, const bf16_t* __restrict__ V,
    bf16_t* __restrict__ O, float* __restrict__ LSE2, int n, int nqb, unsigned nqm, int GQ, int odd,
    int pair_base, int pairs, int rounds, int kv_shift, unsigned kv_magic, float scale_log2e) {
  __shared__ __attribute__((aligned(1024))) char smem[kX2LdsBytes];
  int g0, qb0, vid0 = 0;
  if (rounds > 1) {
    vid0 = (int)(blockIdx.x % 8) * (pairs / 8) + (int)(blockIdx.x / 8);
    g0 = 2 * (vid0 / nqb);
    qb0 = nqb - 1 - vid0 % nqb;
  } else if ((int)blockIdx.x < odd) {
    g0 = GQ - 1;
    qb0 = nqb - 1 - (int)blockIdx.x;
  } else {
    const int per = (pairs + 7) / 8, b = (int)blockIdx.x - odd;
    const int second = b / (8 * per), i = (b % 8) * per + (b % (8 * per)) / 8;
    if (i >= pairs) return;
    const int P = pair_base + i, p = P % nqb;
    const int longer = p < nqb - 1 - p ? 0 : 1;  // of the blocks nqb - 1 - p and p
    const int which = second ^ longer;           // 0: row block nqb - 1 - p of the even head
    g0 = 2 * (P / nqb) + which;
    qb0 = which ? p : nqb - 1 - p;
  }
  g0 = __builtin_amdgcn_readfirstlane(g0);
  qb0 = __builtin_amdgcn_readfirstlane(qb0);
  const int nqbm1 = nqb - 1;

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l32 = lane & 31, h = lane >> 5;
  const unsigned lds0 = (unsigned)(size_t)smem;  // LDS byte address of the stage ring

  // K fragment (16 d-chunk 2kk+h of key row l32): row base and the kk-independent swizzle term
  const unsigned krow = lds0 + l32 * 256, hx16 = (unsigned)((h ^ k_swizzle(l32)) << 4);
  // V fragment (see attn_fwd_kernel): source lane (r, qd) of group gq, key rows 4h + r
  const int i16 = lane & 15, r4 = i16 >> 2, qd = i16 & 3, gq = (lane >> 4) & 1;
  const unsigned clvs16 = (unsigned)(((2 * gq + (qd >> 1)) ^ v_swizzle(r4)) << 4);
  const unsigned vrow = lds0 + kTileBytes + (4 * h + r4) * 256 + (qd & 1) * 8;
  // DMA: this wave fills rows 16u + 4 wave + rr of a tile, lane (rr, pc) the chunk slot pc
  const int rr = lane >> 4, pc = lane & 15, lrow = 4 * wave + rr;
  const unsigned kl0 = (unsigned)(lrow * 256 + ((pc ^ k_swizzle(lrow)) << 4));
  const unsigned vl0 = (unsigned)(lrow * 256 + ((pc ^ v_swizzle(lrow)) << 4));
  const unsigned qoff = (unsigned)(l32 * 256 + h * 16);
  const int lv = l32 - 4 * h;
  const unsigned l32x4 = l32 * 4, lanex16 = lane * 16;
  // epilogue: a wave's 32 x 128 output blocks go, one after the other, through its own 8 KB
  // strip of LDS above the ring
  const unsigned strip = lds0 + kX2RingBytes + wave * 8192;
  const unsigned strip_w = strip + l32 * 256 + 8 * h, x16 = (unsigned)((l32 & 15) << 4);
  const unsigned strip_r = strip + rr * 256, crr16 = (unsigned)((pc ^ rr) << 4);

  // Rows: a 256-row block is cut into eight 32-row blocks; wave w owns blocks w ("block 0")
  // and 7 - w ("block 1"), so that every wave has the same number of key tiles to go through
  // although the rows further down see more keys.
  const int w32a = 32 * wave, w32b = 32 * (7 - wave), wodd = wave & 1;
  const unsigned wave_lds = lds0 + wave * 1024;
  const unsigned long long qa = (unsigned long long)Q, ka = (unsigned long long)K,
                           va = (unsigned long long)V, oa = (unsigned long long)O,
                           la = (unsigned long long)LSE2;

  asm volatile(A2SF_FWD128X2R_ASM
               :
               : [hx16] "v"(hx16), [krow] "v"(krow), [clvs16] "v"(clvs16), [vrow] "v"(vrow),
                 [kl0] "v"(kl0), [vl0] "v"(vl0), [qoff] "v"(qoff), [lv] "v"(lv),
                 [l32x4] "v"(l32x4), [lanex16] "v"(lanex16), [strip_w] "v"(strip_w),
                 [x16] "v"(x16), [crr16] "v"(crr16), [strip_r] "v"(strip_r),
                 [qlo] "s"((unsigned)qa), [qhi] "s"((unsigned)(qa >> 32)),
                 [klo] "s"((unsigned)ka), [khi] "s"((unsigned)(ka >> 32)),
                 [vlo] "s"((unsigned)va), [vhi] "s"((unsigned)(va >> 32)),
                 [olo] "s"((unsigned)oa), [ohi] "s"((unsigned)(oa >> 32)),
                 [llo] "s"((unsigned)la), [lhi] "s"((unsigned)(la >> 32)),
                 [n] "s"(n), [g0] "s"(g0), [qb0] "s"(qb0), [vid0] "s"(vid0), [rounds] "s"(rounds),
                 [nqm] "s"(nqm), [nqbm1] "s"(nqbm1), [w32a] "s"(w32a), [w32b] "s"(w32b),
                 [wodd] "s"(wodd), [wave_lds] "s"(wave_lds), [kvs] "s"(kv_shift), [kvm] "s"(kv_magic),
                 [scale] "s"(scale_log2e)
               : A2SF_FWD128X2R_CLOBBERS);
}

// ---------------------------------------------------------------------------------------
// One workgroup with split keys per compute unit (140 KB of LDS).  As long as every row block has a unit to
// itself, the launch lasts as long as a head's last rows and half the chain is nearly half the time (one
// head x 2000, whole call: 65 -> 43 us; 32 x 1024: 25.0 -> 22.7 in the kernel).  Beyond that, two workgroups
// of four waves per unit share it better (kernel, KS = 1 / 2: 40 heads x 1024 32.1 / 35.4 us, 64 x 1000 34.9 / 42.0,
// 300 x 200 22.4 / 32.3).  Nor for short chains, where the start of the pipeline and the merge cost more (kernel, in turn /
// split: 8 heads x 130 8.1 / 10.4, 8 x 512 13.9 / 13.9, 8 x 900 19.8 / 18.0; d = 64 8 x 130 6.0 / 6.5, 8 x 900 15.6 / 13.4).
constexpr unsigned kSplitKeysMaxBlocks = 256;
constexpr int kSplitKeysMinTiles = 10;
// With d = 128 the pipelined form pays from about 20 tiles on (kernel, in turn / pipelined: 1500 heads x 130 47.8 / 54.8, 300 x
// 900 103 / 104, 96 x 1777 94.3 / 91.9, 600 x 2500 1092 / 1045); with d = 64, where fewer registers let four workgroups
// onto a compute unit, only for the longest (1500 x 130 27.4 / 38.1, 1500 x 900 258 / 325, 96 x 1777 57.3 / 60.1, 40 x 6000 238 /
// 238, 40 x 9000 533 / 513).
template <int D> constexpr int kPipedMinTiles = D == 128 ? 20 : 128;
template <int D>
void launch_fwd_rect(const void* q, const void* k, const void* v, int G, const AttnRect& rc, void* o,
                     float* lse2, hipStream_t st) {
  const float scale_log2e = 1.4426950408889634f / sqrtf((float)D);
  const int GQ = G * rc.kv_group;  // query heads
  constexpr int bm = kWaves * 32;
  const int nqb = (rc.m + bm - 1) / bm - (o ? 0 : rc.first_row / bm);  // row blocks to compute
  const int tiles = ((rc.off_heads ? rc.kv_stride : rc.m) + kTile - 1) / kTile;  // of the newest row, at most
#define A2SF_FWD(WITH_O, KS, PIPED)                                                                   \
  hipLaunchKernelGGL((attn_fwd_kernel<D, WITH_O, KS, PIPED>), dim3(launch_grid<KS == 1 ? kOnePerUnit : kOneRound>(GQ, nqb)), \
                     dim3(kThreads * KS), 0, st, (const bf16_t*)q, (const bf16_t*)k, (const bf16_t*)v, (bf16_t*)o, lse2, rc, \
                     GQ, nqb, scale_log2e)
  if (!o) A2SF_FWD(false, 1, false);
  else if ((long long)GQ * nqb <= kSplitKeysMaxBlocks && tiles >= kSplitKeysMinTiles) A2SF_FWD(true, 2, true);
  else if (tiles >= kPipedMinTiles<D>) A2SF_FWD(true, 1, true);
  else A2SF_FWD(true, 1, false);
#undef A2SF_FWD
}

// Whether attn_fwd128x2r_kernel is the faster one for G heads of n rows.  Both are counted in steps of 256 rows against one
// tile: the pairs of whole double rounds cost every compute unit the same, what is left over lasts as long as one more
// pair (a head's last block and its start, or a longer and a shorter block); a step of the compiled kernel takes 1.2 times
// as long, spread evenly but for its last blocks.  Rows that the last block does not have count in full, so that prompts just
// past a multiple of 256 rows stay with the compiled kernel's blocks of 128 (us, compiled / stream, steps by this count: 1500 heads
// x 513 242 / 312, 107 / 144; 300 x 700 69 / 77, 31 / 32; 1500 x 700 351 / 330, 149 / 144; 1500 x 1000 560 / 514, 255 / 240; 100 x
// 1500 76 / 91, 39 / 56; 300 x 1500 214 / 196, 112 / 112; 50 x 3001 130 / 158, 75 / 104; 128 x 3001 302 / 243, 185 / 156; 100 x 4097
// 435 / 456, 270 / 288; 300 x 4097 1323 / 1275, 796 / 720).
inline bool pair_stream_pays(long long G, int n) {
  const long long nq = (n + kX2Rows - 1) / kX2Rows, nb = (n + kWaves * 32 - 1) / (kWaves * 32), units = 8 * kX2Slots;
  const long long pairs = G / 2 * nq, rest = pairs % units + G % 2 * nq;
  const double stream = (double)((pairs / units + (rest > 0)) * 4 * (nq + 1));
  const double compiled = 1.2 * (double)G * (double)nb * (double)(nb + 1) / (2.0 * (double)units) + 0.2 * (double)nb;
  return stream < compiled;
}

// Square geometry (a whole prompt): G K/V heads, kv_group query heads each.
template <int D>
void launch_fwd(const void* q, const void* k, const void* v, int G_kv, int n, void* o, float* lse2,
                hipStream_t st, int kv_group = 1, int first_row = 0) {
  const float scale_log2e = 1.4426950408889634f / sqrtf((float)D);
  const int G = G_kv * kv_group;  // query heads
  int kv_shift = 0;
  unsigned kv_magic = 0;
  while ((1 << kv_shift) < kv_group) ++kv_shift;
  if ((1 << kv_shift) != kv_group) {   // not a power of two: divide by multiplication
    kv_shift = 31;
    kv_magic = (unsigned)((1ull << 32) / (unsigned)kv_group) + 1u;
  }
  if constexpr (D == 128) {
    // Two query blocks per wave pay off from n = 512 on in the persistent form, which overlaps the start and the
    // end of a row block with its neighbours.
    // Few row blocks: the split keys of attn_fwd_kernel<.., 2> shorten the longest chain of tiles
    // (8 heads x 4096, whole call: 122.6 us here, 73.5 there).
    const bool few = (long long)G * ((n + kWaves * 32 - 1) / (kWaves * 32)) <= kSplitKeysMaxBlocks;
    if (o && !few && n >= kX2MinRows && (long long)G * n < (1ll << 31)) {
      const int nqb2 = (n + kX2Rows - 1) / kX2Rows;
      const long long items = (long long)G * nqb2;
      const int chunk = 2 * 8 * kX2Slots;  // items of two rounds of the persistent launch
      const bool persistent = items >= chunk && items < (1ll << 31);
      // whole row blocks whose number divides a round: ids are split by shifts
      const bool aligned = n % kX2Rows == 0 && (nqb2 & (nqb2 - 1)) == 0 && nqb2 <= kX2Slots;
      if (persistent && aligned) {
        auto launch = [&](int id_base, int ids, int rounds) {
          const unsigned grid2 = rounds > 1 ? 8 * kX2Slots : (unsigned)(((ids + 7) / 8) * 8);
          hipLaunchKernelGGL(attn_fwd128x2_kernel, dim3(grid2), dim3(kThreads), 0, st,
                             (const bf16_t*)q, (const bf16_t*)k, (const bf16_t*)v, (bf16_t*)o, lse2, n,
                             nqb2, id_base, ids, rounds, kv_shift, kv_magic, scale_log2e);
        };
        // persistent part: an even number of full rounds; what is left over goes one workgroup
        // per row block
        const int main_ids = (int)(items / chunk) * chunk;
        launch(0, main_ids, main_ids / (8 * kX2Slots));
        if (items > main_ids) launch(main_ids, (int)(items - main_ids), 1);
        return;
      }
      if (pair_stream_pays(G, n)) {
        const unsigned nqm = (unsigned)((1ull << 32) / (unsigned)nqb2) + 1u;  // exact below 2^32 / nqb2
        const int all = (G / 2) * nqb2, odd = (G % 2) * nqb2;
        auto launch = [&](int odd_blocks, int base, int pairs, int rounds) {
          const unsigned grid2 = rounds > 1 ? 8 * kX2Slots : (unsigned)(odd_blocks + 16 * ((pairs + 7) / 8));
          hipLaunchKernelGGL(attn_fwd128x2r_kernel, dim3(grid2), dim3(kThreads), 0, st, (const bf16_t*)q,
                             (const bf16_t*)k, (const bf16_t*)v, (bf16_t*)o, lse2, n, nqb2, nqm, G, odd_blocks,
                             base, pairs, rounds, kv_shift, kv_magic, scale_log2e);
        };
        // pairs of whole double rounds in the persistent form (its ids stay below 2^32 / nqb2: n < 2^24)
        const int main_pairs = (long long)all * nqb2 < (1ll << 32) ? all / (8 * kX2Slots) * (8 * kX2Slots) : 0;
        if (main_pairs) launch(0, 0, main_pairs, main_pairs / (4 * kX2Slots));
        if (odd || all > main_pairs) launch(odd, main_pairs, all - main_pairs, 1);
        return;
      }
    }
  }
  // Without outputs the pass is bound by the vector ALU as much as by the matrix cores
  // (fma + exp + add per logit against 1/16 matrix op): one 32-row block per wave at four
  // workgroups per compute unit overlaps the two better than two blocks per wave at two
  // (16384 heads of n = 2048: 11.1 ms against 12.75 when both forms were there; 9.6 in the form without the pipeline).
  AttnRect rc{n, n, nullptr, kv_group};
  rc.first_row = o ? 0 : first_row;
  launch_fwd_rect<D>(q, k, v, G_kv, rc, o, lse2, st);
}

// ---------------------------------------------------------------------------------------
// col_scores for a short row window (alpha well below 1).  Only rows >= first_row
// contribute (see first_contributing_row), at most kTailTiles tiles of 64 rows.  One
// workgroup per head (with few heads: per share of a head's keys) stages those Q rows in LDS
// once (direct global-to-LDS loads) and then walks over its key blocks: a wave keeps 32 keys
// as A fragments in registers (the next block's fragments are fetched while the current block
// is computed), recomputes the logit tiles against the staged Q rows, applies
// exp2(s - lse_i + (n-1-i) log2 alpha) and sums down the rows.  K is read exactly once, Q's
// window once per workgroup.
constexpr int kTailTiles = 4;
constexpr int kTailKB = 2;  // 32-key blocks per wave and step

// Row window for a relative tolerance on the scores (Section 3.3: the forgetting factor makes
// old rows' contributions go to 0).  All rows before n - W together add at most
// alpha^W / (1 - alpha) to any S_j (probabilities are <= 1), while S_j >= P[n-1, j]; so for a
// group of keys whose smallest P[n-1, j] is p_min every S_j of the group is exact to a
// relative `tol` once  alpha^W <= tol (1 - alpha) p_min.  p_min is read off the newest row,
// which a wave processes first; zmin is log2 of the probabilities a lane saw there.
struct RowWindow {
  bool on;
  float tl2, inv_l2a;
  __device__ RowWindow(float tol, float log2_alpha) {
    on = tol > 0.f && log2_alpha < 0.f;
    tl2 = on ? log2f(tol * (1.f - exp2f(log2_alpha))) : 0.f;
    inv_l2a = on ? 1.f / log2_alpha : 0.f;
  }
  // first row a wave has to process; zmin as held by the lanes `lane_last` and `lane_last + 32`
  // (the two halves of the newest row)
  __device__ __forceinline__ int first_row(int n, float zmin, int lane_last) const {
    const float z0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(zmin), lane_last));
    const float z1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(zmin), lane_last + 32));
    const float need = (tl2 + fminf(z0, z1)) * inv_l2a;   // rows needed (both factors negative)
    return need >= (float)n ? 0 : n - ((int)need + 2);
  }
};

template <int D>
__global__ __launch_bounds__(kThreads, 2) void col_scores_tail_kernel(
    const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, const float* __restrict__ LSE2,
    float* __restrict__ S, AttnRect rc, int s_stride, bool accumulate, float decay, int first_row,
    float log2_alpha, const float* __restrict__ alpha_heads, float scale_log2e, float tol, int ksplit) {
  constexpr int KK = D / 16, BC = kWaves * 32, kTB = kTileBytesOf<D>;
  __shared__ __attribute__((aligned(1024))) char smem[kTailTiles * kTB];
  __shared__ __attribute__((aligned(16))) float strip[kWaves][32 * kTailKB];   // a wave's scores of one step
  lds_char* const qs = (lds_char*)smem;

  // ksplit workgroups share a head's keys (few heads with long prompts: one workgroup per head
  // would leave most of the chip idle); each stages the row window for itself
  const int g = blockIdx.x / ksplit, kpart = blockIdx.x % ksplit;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform: branches on it are scalar
  const int l32 = lane & 31, h = lane >> 5;
  // n query rows; row i sees keys 0 .. off + i of the head's nk = off + n keys (the prompt
  // phase: off = 0; a chunk of a prompt: off = tokens cached before it)
  const int n = rc.m;
  const int off = rect_off(rc, g);
  if (off < 0) return;  // a head the caller's precondition excludes
  const int nk = off + n;
  constexpr int STEP = BC * kTailKB;  // keys per workgroup step
  const int kspan = ((nk + ksplit * STEP - 1) / (ksplit * STEP)) * STEP;  // keys per workgroup
  const int c_begin = kpart * kspan, c_end = min(nk, c_begin + kspan);
  if (c_begin >= nk) return;
  const bf16_t* Qg = Q + (size_t)g * n * D;
  const bf16_t* Kg = K + (size_t)g * rc.kv_stride * D;
  const bf16_t* K2g = rc.k2 ? (const bf16_t*)rc.k2 + (size_t)g * n * D : nullptr;  // keys off .. from here
  const float* lse = LSE2 + (size_t)g * n;
  float* Sg = S + (size_t)g * s_stride;

  const int r_lo = (first_row / kTile) * kTile;          // first staged row (sized by the host)
  head_window(alpha_heads, g, n, first_row, log2_alpha);  // this head's own window inside it
  const int ntile = (n - r_lo + kTile - 1) / kTile;      // <= kTailTiles (checked by the host)
#pragma unroll
  for (int tt = 0; tt < kTailTiles; ++tt)
    if (tt < ntile) dma_tile<D, false>(Qg, r_lo + tt * kTile, n, qs + tt * kTB);

  int qoff[KK];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) qoff[kk] = l32 * D * 2 + (((2 * kk + h) ^ k_swizzle<D>(l32)) << 4);
  // exponent offset of this lane's row in each 32-row block: lse_i - (n-1-i) log2 alpha;
  // +inf (probability 0) for rows past the end or before the window
  // (all loads issued before the first is used: the address is clamped, not the load skipped)
  float bias[2 * kTailTiles];
#pragma unroll
  for (int rb = 0; rb < 2 * kTailTiles; ++rb) bias[rb] = lse[min(r_lo + rb * 32 + l32, n - 1)];
#pragma unroll
  for (int rb = 0; rb < 2 * kTailTiles; ++rb) {
    const int r = r_lo + rb * 32 + l32;
    bias[rb] = (r < n && r >= first_row) ? bias[rb] - (float)(n - 1 - r) * log2_alpha : INFINITY;
  }
  // A wave owns kTailKB blocks of 32 keys at a time: every Q fragment read from LDS feeds
  // kTailKB matrix ops (one LDS kilobyte per matrix op is more than the LDS delivers).
  auto load_keys = [&](int c0, uint4 (&kf)[kTailKB][KK]) {
#pragma unroll
    for (int b = 0; b < kTailKB; ++b) {
      int r = c0 + (wave * kTailKB + b) * 32 + l32;
      r = r < nk ? r : nk - 1;
      const bf16_t* row = (K2g && r >= off) ? K2g + (size_t)(r - off) * D : Kg + (size_t)r * D;
#pragma unroll
      // (plain loads: a lane takes 32 bytes of its key's row per instruction, so every 128-byte
      // line is shared by four instructions and has to stay in the cache between them)
      for (int kk = 0; kk < KK; ++kk) kf[b][kk] = load16(row + kk * 16 + h * 8);
    }
  };
  uint4 kf[kTailKB][KK];
  load_keys(c_begin, kf);
  wait_vm_barrier<0>();  // the staged rows of every wave

  const RowWindow win(tol, log2_alpha);
  const int rb_last = (n - 1 - r_lo) >> 5;   // the row block that holds the newest row
  const int lane_last = (n - 1 - r_lo) & 31;
  for (int c0 = c_begin; c0 < c_end; c0 += STEP) {
    const int wc0 = c0 + wave * kTailKB * 32;  // first key of this wave in this step
    int lim = max(wc0 - off, first_row);       // rows before `lim` add nothing to this wave's keys
    bool pending = c0 + STEP < c_end;          // the next step's keys still have to be fetched
    float acc[kTailKB][16];
#pragma unroll
    for (int b = 0; b < kTailKB; ++b)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[b][i] = 0.f;
    // newest rows first: the block of the last row tells how far back this wave has to go
#pragma unroll
    for (int rb = 2 * kTailTiles - 1; rb >= 0; --rb) {
      const int rr0 = r_lo + rb * 32;
      if (rb <= rb_last && rr0 + 31 >= lim) {  // wave-uniform
        f32x16 sacc[kTailKB];
#pragma unroll
        for (int b = 0; b < kTailKB; ++b)
#pragma unroll
          for (int i = 0; i < 16; ++i) sacc[b][i] = 0.f;
        const lds_char* qt = qs + rb * 32 * D * 2;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
          const uint4 qf = lds_read16(qt + qoff[kk]);
#pragma unroll
          for (int b = 0; b < kTailKB; ++b) sacc[b] = mfma_bf16(kf[b][kk], qf, sacc[b]);
        }
        // last use of kf is behind us once no older row block follows
        if (pending && rb != rb_last && (rb == 0 || rr0 - 1 < lim)) {
          load_keys(c0 + STEP, kf);
          pending = false;
        }
        const int r = rr0 + l32;
        if (win.on && rb == rb_last) {   // log2 of the newest row's smallest probability, per lane
          float zmin = INFINITY;
#pragma unroll
          for (int b = 0; b < kTailKB; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) zmin = fminf(zmin, fmaf(sacc[b][i], scale_log2e, -bias[rb]));
          lim = max(lim, win.first_row(n, zmin, lane_last));
        }
#pragma unroll
        for (int b = 0; b < kTailKB; ++b) {
          const int bk0 = wc0 + b * 32;
          if (bk0 + 31 > off + rr0) {  // block touches the diagonal: keys above the row contribute 0
#pragma unroll
            for (int i = 0; i < 16; ++i) {
              const int key = bk0 + 8 * (i >> 2) + 4 * h + (i & 3);
              const float p = fast_exp2(fmaf(sacc[b][i], scale_log2e, -bias[rb]));
              acc[b][i] += key > off + r ? 0.f : p;
            }
          } else {
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[b][i] += fast_exp2(fmaf(sacc[b][i], scale_log2e, -bias[rb]));
          }
        }
      }
    }
    if (pending) load_keys(c0 + STEP, kf);
    // sum over the 32 rows held by the lanes of one half; the wave's 32 * kTailKB scores go
    // through its LDS strip so that they leave as whole 16-byte pieces of one contiguous run
    // (two lanes hold them all, four consecutive keys per register quad)
#pragma unroll
    for (int b = 0; b < kTailKB; ++b) {
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[b][i] = group_sum<32>(acc[b][i]);
      if (l32 == 0) {
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4)   // keys b*32 + 8*i4 + 4h .. +3
          *reinterpret_cast<float4*>(&strip[wave][b * 32 + 8 * i4 + 4 * h]) =
              make_float4(acc[b][4 * i4], acc[b][4 * i4 + 1], acc[b][4 * i4 + 2], acc[b][4 * i4 + 3]);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    __builtin_amdgcn_wave_barrier();
    if (lane < 8 * kTailKB) {
      const int key = wc0 + 4 * lane;
      float4 v = *reinterpret_cast<const float4*>(&strip[wave][4 * lane]);
      float* out = Sg + key;
      // `accumulate`: on top of `decay` times the older score (a chunk: alpha^n); the chunk's own keys have none
      const float vv[4] = {v.x, v.y, v.z, v.w};
      if (key + 3 < nk && (reinterpret_cast<size_t>(out) & 15) == 0) {
        if (accumulate) {
          const float4 old = *reinterpret_cast<const float4*>(out);
          const float ov[4] = {old.x, old.y, old.z, old.w};
          float sum[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) sum[e] = key + e < off ? fmaf(decay, ov[e], vv[e]) : vv[e];
          v = make_float4(sum[0], sum[1], sum[2], sum[3]);
        }
        *reinterpret_cast<float4*>(out) = v;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (key + e < nk) out[e] = accumulate && key + e < off ? fmaf(decay, out[e], vv[e]) : vv[e];
      }
      if (rc.pos) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (key + e >= off && key + e < nk) rc.pos[(size_t)g * rc.kv_stride + key + e] = rc.pos0 + key + e - off;
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    __builtin_amdgcn_wave_barrier();   // the strip is rewritten in the next step
  }
}

// ---------------------------------------------------------------------------------------
// col_scores for a long row window (alpha close to 1), for grouped-query heads and for few keys: the
// streaming form of col_scores_tail_kernel.  A workgroup owns 128 key columns (a wave KB = 1 block of 32
// keys, or 256 columns and KB = 2, the K fragments resident in registers for the whole kernel) and walks down the rows that
// see them, one query head of the group after the other; Q tiles of 64 rows arrive by direct
// global-to-LDS loads in a ring, one tile (KB = 2: three tiles) ahead of the one being used.  One barrier
// per tile publishes the tile that has landed and frees the stage of the previous one for the next fetch.
// One block and two stages leave room for four workgroups per compute unit, which hide the loads and the vector work (the
// exponentials) better than two blocks that share a Q fragment and a ring of four (us, alpha = 1, KB = 2 / 1: 300 heads x 260
// 25 / 16, 300 x 1000 82 / 66, 96 x 1777 63 / 57, 300 x 4000 796 / 774; d = 64, 96 x 1777 52 / 42).  But they read the rows twice as
// often, and from about 8000 rows on a die's heads do not stay in its L2 (64 x 9000 749 / 783; d = 64 never minds).
// Geometry as in AttnRect (n = rc.m rows, keys 0 .. off + n - 1, row i sees keys <= off + i).
// accumulate: the column sums are added to decay * S[] for the keys before off (a chunk: the cached tokens' older
// scores decayed by alpha^m) instead of replacing it.
// RS = 2, 4 (without a tolerance): 4 RS waves, of which four take every RS-th tile for the same keys, each
// part with a ring of its own; their sums meet at the end.  For launches whose workgroups are all
// resident at once, which last as long as the column block with the most rows.
template <int D, int KB, int RS>
__global__ __launch_bounds__(kThreads * RS, (KB == 1 ? 4 : 2) / RS) void col_scores_stream_kernel(
    const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, const float* __restrict__ LSE2,
    float* __restrict__ S, AttnRect rc, int s_stride, bool accumulate, float decay, int G, int ncb, int first_row,
    float log2_alpha, const float* __restrict__ alpha_heads, float scale_log2e, float tol) {
  constexpr int KK = D / 16, BC = kWaves * 32 * KB, kTB = kTileBytesOf<D>, kStages = KB == 1 ? 2 : 4;
  constexpr int NL = kLoadsPerWave<D>, kLoads = NL + 1;  // loads of a wave per tile
  // Q tiles, then per wave and stage the 64 log-sum-exp values of the tile's rows
  constexpr int kLds = kStages * kTB + kWaves * kStages * 256;
  __shared__ __attribute__((aligned(1024))) char smem[RS * kLds];
  __shared__ int wave_lim[kWaves];
  __shared__ float other[RS > 1 ? RS - 1 : 1][RS > 1 ? BC : 1];

  int g, cb;  // column block 0 has the most rows
  if (!launch_item<RS == 1 ? kTwoPerUnit : kOneRound>(G, ncb, g, cb)) return;
  const int n = rc.m;
  const int off = rect_off(rc, g);
  const int nk = off + n;  // keys of this head
  const int c0 = cb * BC;
  if (off < 0 || c0 >= nk) return;
  head_window(alpha_heads, g, n, first_row, log2_alpha);

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6) % kWaves;  // wave-uniform: branches on it are scalar
  const int part = RS > 1 ? __builtin_amdgcn_readfirstlane(tid >> 6) / kWaves : 0;
  lds_char* const qs = (lds_char*)smem + part * kLds;
  const int l32 = lane & 31, h = lane >> 5;
  const bf16_t* Qg = Q + (size_t)g * rc.kv_group * n * D;  // the group's rows lie one head after the other
  const bf16_t* Kg = K + (size_t)g * rc.kv_stride * D;
  const bf16_t* K2g = rc.k2 ? (const bf16_t*)rc.k2 + (size_t)g * n * D : nullptr;  // keys off .. from here
  const float* lse = LSE2 + (size_t)g * rc.kv_group * n;
  const int wc0 = c0 + wave * 32 * KB;  // first key of this wave

  // Tiles are walked from the newest rows down: with a tolerance (one query head per K/V head) the
  // newest row tells how far back the workgroup has to go (RowWindow), and without one the order
  // does not matter.
  const int t_last = (n + kTile - 1) / kTile - 1;
  int t_first = max(max(c0 - off, first_row), 0) / kTile;  // oldest tile any wave of the workgroup needs
  lds_char* const lse_s = qs + kStages * kTB + wave * (kStages * 256);
  // tile f of the sequence is tile t_last - f % per_head of query head f / per_head; this part takes
  // the tiles part, part + RS, ...
  int per_head = t_last - t_first + 1;
  // The part's next Q tile into the next ring stage (every wave a quarter of the rows) and the rows'
  // log-sum-exp values into the wave's own strip of that stage; always issued (past the last tile the
  // last one again, never used), so that the wait counts in the loop are the same for every tile.
  int f_hq = 0, f_i = part, f_stage = 0;  // query head and place in its sequence of the next fetch
  int f_loff[NL];
  dma_offsets<D, false>(f_loff);
  auto fetch = [&]() {
    while (f_i >= per_head) {
      if (f_hq + 1 < rc.kv_group) { ++f_hq; f_i -= per_head; }
      else f_i = per_head - 1;
    }
    const size_t head = (size_t)f_hq * n;
    const int row0 = (t_last - f_i) * kTile;
    if (row0 + kTile <= n) dma_full_tile<D>(Qg + head * D, row0, f_loff, qs + f_stage * kTB);
    else dma_tile<D, false>(Qg + head * D, row0, n, qs + f_stage * kTB);
    dma4(lse + head + row0, (uint32_t)(min(lane, n - 1 - row0) * 4), (uint32_t)(size_t)(lse_s + f_stage * 256));
    f_stage = (f_stage + 1) % kStages;
    f_i += RS;
  };
#pragma unroll
  for (int i = 1; i < kStages; ++i) fetch();

  // K fragments (A operand): lane (key l32, half h) holds K[key][16kk + 8h .. +7]
  uint4 kf[KB][KK];
#pragma unroll
  for (int b = 0; b < KB; ++b) {
    const int r = min(wc0 + b * 32 + l32, nk - 1);
    const bf16_t* row = (K2g && r >= off) ? K2g + (size_t)(r - off) * D : Kg + (size_t)r * D;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) kf[b][kk] = load16(row + kk * 16 + h * 8);
  }
  int qoff[KK];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) qoff[kk] = l32 * D * 2 + (((2 * kk + h) ^ k_swizzle<D>(l32)) << 4);
  float acc[KB][16];
#pragma unroll
  for (int b = 0; b < KB; ++b)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[b][i] = 0.f;

#pragma unroll
  for (int b = 0; b < KB; ++b)
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) asm volatile("" : "+v"(kf[b][kk].x));  // waited for here, not in the loop
  const RowWindow win(tol, log2_alpha);
  int lim = max(wc0 - off, first_row);   // rows before `lim` add nothing to this wave's keys
  int stage = 0, i_seq = part;
  const int steps = (rc.kv_group * per_head + RS - 1) / RS;
  for (int u = 0; u < steps; ++u, stage = (stage + 1) % kStages, i_seq += RS) {
    while (i_seq >= per_head) i_seq -= per_head;
    const int t = t_last - i_seq;
    const bool own = RS == 1 || u * RS + part < rc.kv_group * per_head;  // (a part may be one tile short)
    // this tile has landed: of this wave's fetches only those of the tiles behind it may still be under way
    wait_vm_barrier<(kStages - 2) * kLoads>();
    fetch();  // into the stage of the previous tile, which every wave has left
    const int row0 = t * kTile;
    if (own && row0 + kTile - 1 >= lim) {  // some row of the tile counts for a key of this wave
      const lds_char* qt = qs + stage * kTB;
      const __attribute__((address_space(3))) float* lse_t =
          (const __attribute__((address_space(3))) float*)(lse_s + stage * 256);
      float zmin[2] = {INFINITY, INFINITY};
#pragma unroll
      for (int qb = 1; qb >= 0; --qb) {
        f32x16 sacc[KB];
#pragma unroll
        for (int b = 0; b < KB; ++b)
#pragma unroll
          for (int i = 0; i < 16; ++i) sacc[b][i] = 0.f;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
          const uint4 qf = lds_read16(qt + qb * 32 * D * 2 + qoff[kk]);
#pragma unroll
          for (int b = 0; b < KB; ++b) sacc[b] = mfma_bf16(kf[b][kk], qf, sacc[b]);
        }
        const int r = row0 + qb * 32 + l32;
        // exponent offset of row r: lse_r - (n-1-r) log2(alpha); rows past the end, and rows
        // whose weight is exactly 0 in fp32 (before first_row), add nothing
        const float bias = (r < n && r >= first_row)
                               ? lse_t[qb * 32 + l32] - (float)(n - 1 - r) * log2_alpha : INFINITY;
        if (win.on && t == t_last) {   // log2 of the newest row's smallest probability, per lane
          float zm = INFINITY;
#pragma unroll
          for (int b = 0; b < KB; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) zm = fminf(zm, fmaf(sacc[b][i], scale_log2e, -bias));
          zmin[qb] = zm;
        }
#pragma unroll
        for (int b = 0; b < KB; ++b) {
          const int bk0 = wc0 + b * 32;
          if (bk0 + 31 > off + row0 + qb * 32) {  // block reaches above the diagonal
#pragma unroll
            for (int i = 0; i < 16; ++i) {
              const int key = bk0 + 8 * (i >> 2) + 4 * h + (i & 3);
              const float p = fast_exp2(fmaf(sacc[b][i], scale_log2e, -bias));
              acc[b][i] += key > off + r ? 0.f : p;
            }
          } else {
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[b][i] += fast_exp2(fmaf(sacc[b][i], scale_log2e, -bias));
          }
        }
      }
      if (win.on && t == t_last) {
        const int rl = n - 1 - row0;   // the newest row inside this tile
        lim = max(lim, win.first_row(n, rl >= 32 ? zmin[1] : zmin[0], rl & 31));
      }
    }
    if (win.on && t == t_last) {   // the workgroup stops at the oldest tile one of its waves needs
      if (lane == 0) wave_lim[wave] = lim;
      __syncthreads();
      const int wl = min(min(wave_lim[0], wave_lim[1]), min(wave_lim[2], wave_lim[3]));
      t_first = max(t_first, wl / kTile);
      per_head = t_last - t_first + 1;
      if (per_head <= 1) break;
    }
    if (win.on && t <= t_first) break;
  }
  wait_vm<0>();  // tiles fetched ahead of the last one used: let them land
  // sum over the 32 rows held by the lanes of one half, then over the parts of the workgroup
#pragma unroll
  for (int b = 0; b < KB; ++b)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[b][i] = group_sum<32>(acc[b][i]);
  // Every lane of a half has the half's 16 sums per block; sixteen of them take one each, so that the scores leave in one store.
  float sum[KB];
#pragma unroll
  for (int b = 0; b < KB; ++b) {
    sum[b] = acc[b][0];
#pragma unroll
    for (int i = 1; i < 16; ++i) sum[b] = (lane & 15) == i ? acc[b][i] : sum[b];
  }
  const int key_l = 8 * ((lane & 15) >> 2) + 4 * h + (lane & 3), w0 = wave * 32 * KB;
  if constexpr (RS > 1) {
    if (part > 0 && l32 < 16) {
#pragma unroll
      for (int b = 0; b < KB; ++b) other[part - 1][w0 + b * 32 + key_l] = sum[b];
    }
    __syncthreads();
    if (part > 0) return;
  }
  if (l32 >= 16) return;
#pragma unroll
  for (int b = 0; b < KB; ++b) {
    const int key = wc0 + b * 32 + key_l;
    if (key >= nk) continue;
    float x = sum[b];
#pragma unroll
    for (int p = 1; p < RS; ++p) x += other[p - 1][w0 + b * 32 + key_l];
    float* out = S + (size_t)g * s_stride + key;
    *out = accumulate && key < off ? fmaf(decay, *out, x) : x;
    if (rc.pos && key >= off) rc.pos[(size_t)g * rc.kv_stride + key] = rc.pos0 + key - off;
  }
}

// ---------------------------------------------------------------------------------------
// Scores, selection and moves of a short prompt or chunk in one kernel, one workgroup per K/V head: three launches
// whose work is a few chains of latencies.  Up to 256 rows that count and KEYS keys: KEYS / 32 waves (of four at least) have a block of 32 keys each in
// registers, the rows are staged in LDS as in col_scores_tail_kernel, one query head of the group after the other; the
// scores stay in LDS, where one wave selects from them.  (The exponent offsets are in LDS and the loop over the rows is not
// unrolled: such a kernel runs once per compute unit, and its instructions have to be fetched first.)
// MOVE: kGather, a prompt; kInPlace, a chunk, whose new tokens' positions are rc.pos0 ... (K is then the cache, whose rows change: it
// is not a restricted argument).
constexpr int kScoreSelectKeys = 512;  // largest form
template <int KEYS> constexpr int kScoreSelectThreads = KEYS < kThreads / 2 ? kThreads : 2 * KEYS;
template <int D, int MOVE, int KEYS>
__global__ __launch_bounds__(kScoreSelectThreads<KEYS>) void scores_select_kernel(
    const bf16_t* __restrict__ Q, const bf16_t* K, const float* __restrict__ LSE2, AttnRect rc, float decay,
    int first_row, float log2_alpha, const float* __restrict__ alpha_heads, float scale_log2e, float* __restrict__ scores_full,
    int select, int recent, MoveTo to) {
  constexpr int T = kScoreSelectThreads<KEYS>, KK = D / 16, kTB = kTileBytesOf<D>;
  constexpr int TILES = KEYS < kTailTiles * kTile ? KEYS / kTile : kTailTiles;  // (no more rows than keys)
  __shared__ __attribute__((aligned(1024))) char smem[TILES * kTB];
  __shared__ float bias[TILES * kTile], z[KEYS];
  __shared__ int32_t list[KEYS];
  __shared__ SelectSmem<1> none;
  lds_char* const qs = (lds_char*)smem;
  const int g = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, h = lane >> 5;
  const int n = rc.m;
  const int off = rect_off(rc, g);
  if (off < 0) return;  // a head the caller's precondition excludes
  const int nk = off + n;  // <= KEYS (checked by the host)
  const bf16_t* K2g = rc.k2 ? (const bf16_t*)rc.k2 + (size_t)g * n * D : nullptr;  // keys off .. from here
  const int r_lo = (first_row / kTile) * kTile;           // first staged row (sized by the host)
  head_window(alpha_heads, g, n, first_row, log2_alpha);  // this head's own window inside it
  const int ntile = (n - r_lo + kTile - 1) / kTile;       // <= TILES (checked by the host)
  uint4 kf[KK];  // A operand: lane (key l32, half h) holds K[key][16kk + 8h .. +7]
  {
    const int r = min(wave * 32 + l32, nk - 1);
    const bf16_t* row = (K2g && r >= off) ? K2g + (size_t)(r - off) * D : K + ((size_t)g * rc.kv_stride + r) * D;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) kf[kk] = load16(row + kk * 16 + h * 8);
  }
  int qoff[KK];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) qoff[kk] = l32 * D * 2 + (((2 * kk + h) ^ k_swizzle<D>(l32)) << 4);
  const int rb_last = (n - 1 - r_lo) >> 5;  // the row block that holds the newest row
  const int lim = max(wave * 32 - off, first_row);  // rows before `lim` add nothing to this wave's keys
  const int rb_first = max(lim - r_lo, 0) >> 5;
  float acc[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = 0.f;
  for (int hq = 0; hq < rc.kv_group; ++hq) {
    const size_t head = (size_t)g * rc.kv_group + hq;
    if (hq > 0) __syncthreads();  // every wave is done with the rows of the head before
    for (int t = wave / kWaves; t < ntile; t += T / kThreads) dma_tile<D, false>(Q + head * n * D, r_lo + t * kTile, n, qs + t * kTB);
    // exponent offset of every staged row: lse_r - (n-1-r) log2 alpha, infinite where it adds nothing
    if (tid < TILES * kTile) {
      const int r = r_lo + tid;
      const float lse = LSE2[head * n + min(r, n - 1)];
      bias[tid] = (r < n && r >= first_row) ? lse - (float)(n - 1 - r) * log2_alpha : INFINITY;
    }
    wait_vm_barrier<0>();
    if (wave * 32 < nk) {
#pragma unroll 1
      for (int rb = rb_first; rb <= rb_last; ++rb) {
        f32x16 s;
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] = 0.f;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) s = mfma_bf16(kf[kk], lds_read16(qs + rb * 32 * D * 2 + qoff[kk]), s);
        const float b = bias[rb * 32 + l32];
        const int newest = off + r_lo + rb * 32 + l32;  // newest key this lane's row sees
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const float p = fast_exp2(fmaf(s[i], scale_log2e, -b));
          acc[i] += wave * 32 + 8 * (i >> 2) + 4 * h + (i & 3) > newest ? 0.f : p;
        }
      }
    }
  }
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = group_sum<32>(acc[i]);
  float sum = acc[0];
#pragma unroll
  for (int i = 1; i < 16; ++i) sum = (lane & 15) == i ? acc[i] : sum;
  const int key = wave * 32 + 8 * ((lane & 15) >> 2) + 4 * h + (lane & 3);
  if (l32 < 16 && key < nk) {
    if (MOVE == kInPlace && key < off) sum = fmaf(decay, to.s[(size_t)g * to.capacity + key], sum);
    z[key] = sum;
    if (scores_full) scores_full[(size_t)g * n + key] = sum;
  }
  __syncthreads();
  const int B = select + recent, kept = min(nk, B);
  const auto score = [&](int j) { return z[j]; };
  const auto position = [&](int j) {
    return MOVE == kGather ? j : (j < off ? to.p[(size_t)g * to.capacity + j] : rc.pos0 + j - off);
  };
  if (nk <= B) {
    if (tid < nk) list[tid] = tid;
  } else if (wave == 0) {
    select_slots<1, KEYS / kWave>(score, position, MOVE == kInPlace, nk, select, recent, 0, list, none);
  }
  __syncthreads();
  if (tid == 0) to.len[g] = kept;
  if constexpr (MOVE == kInPlace) move_rows<T>(to, list, kept, g, off, true, score, position);
  else gather_rows<T>(to, list, kept, g, n, score);
}

// Workgroups per head of col_scores_tail_kernel: with fewer heads than the chip takes
// workgroups (two per compute unit), a head's keys are shared out, in steps of 256 keys.
inline int tail_key_split(int G, int keys_per_head) {
  const int steps = (keys_per_head + kWaves * 32 * kTailKB - 1) / (kWaves * 32 * kTailKB);
  const int want = (512 + G - 1) / G;
  return want < 1 ? 1 : (want > steps ? steps : want);
}

// Rows split over the two halves of a workgroup of col_scores_stream_kernel: while every workgroup has a compute unit to
// itself and at least four tiles, or half a unit and sixteen (us, alpha = 1, four waves / eight: one head x 1000 20.8 /
// 15.2, 40 x 640 15.5 / 12.9, 100 groups of 4 x 130 18.9 / 15.2, 40 x 1000, 320 blocks, 26.2 / 24.9, but 100 x 130, three
// tiles, 8.3 / 9.4 and 100 x 400, 400 blocks, 15.1 / 19.9); beyond that the halves wait for each other (300 x 1000 66 / 113).
constexpr unsigned kStreamSplitMaxBlocks = 256;
constexpr int kStreamSplitMinTiles = 4;
// In four parts: the chain of a tile (products, exponentials, sums: 1.2 us for a wave that shares its SIMD with one other)
// counts, not the loads: deeper rings make no difference (us, two parts / four: d = 64, one head x 1000, 16 tiles, 12.9 / 12.0, x 4000
// 40.4 / 31.6, one group of 8 x 1000 78 / 60, 240 blocks of 4 x 16 tiles 43.2 / 35.0, but 9 tiles 9.2 / 9.6; d = 128, one head
// x 4000 44.4 / 38.7, one group of 8 x 1000 85 / 72, 24 tiles 22.0 / 20.3, 20 18.7 / 18.8, 16 15.3 / 16.0).
template <int D> constexpr int kStreamFourMinTiles = D == 64 ? 12 : 24;
// KB = 2, d = 128: see above, and with two wide blocks per unit (8 x 9000, KB = 2 / 1: 223 / 173, 16 x 16000 588 / 617).
constexpr int kStreamWideMinTiles = 128, kStreamWideMinBlocks = 1024;
// Up to one block of keys the staging of col_scores_tail_kernel does not pay (1000 heads x 100, streamed / staged: 13.7 / 19.2 us,
// d = 64 10.2 / 13.1; 200 keys: 25 / 28, 20.6 / 18.7).
constexpr int kTailMinKeys = 128;

// Column scores for any head size and geometry.
template <int D>
void launch_cols(const void* q, const void* k, const float* lse2, int G, const AttnRect& rc,
                 int keys_per_head, float alpha, const float* alpha_heads, float tol, float* scores,
                 int s_stride, bool accumulate, float decay, hipStream_t st) {
  const float scale_log2e = 1.4426950408889634f / sqrtf((float)D);
  float l2a;
  const int first = first_contributing_row(rc.m, alpha, &l2a);
  // one query head per K/V head and a row window of at most four tiles: staged once per head,
  // every key streamed once
  if (rc.kv_group == 1 && keys_per_head > kTailMinKeys && rc.m - (first / kTile) * kTile <= kTailTiles * kTile) {
    const int ks = tail_key_split(G, keys_per_head);
    hipLaunchKernelGGL((col_scores_tail_kernel<D>), dim3(G * ks), dim3(kThreads), 0, st, (const bf16_t*)q,
                       (const bf16_t*)k, lse2, scores, rc, s_stride, accumulate, decay, first, l2a,
                       alpha_heads, scale_log2e, tol, ks);
    return;
  }
#define A2SF_STREAM(KB, RS)                                                                           \
  do {                                                                                                \
    const int ncb = (keys_per_head + kWaves * 32 * KB - 1) / (kWaves * 32 * KB);                      \
    hipLaunchKernelGGL((col_scores_stream_kernel<D, KB, RS>), dim3(launch_grid<RS == 1 ? kTwoPerUnit : kOneRound>(G, ncb)), \
                       dim3(kThreads * RS), 0, st, (const bf16_t*)q, (const bf16_t*)k, lse2, scores, rc, s_stride, \
                       accumulate, decay, G, ncb, first, l2a, alpha_heads, scale_log2e, tol);         \
  } while (0)
  const int tiles = (rc.m + kTile - 1) / kTile - first / kTile;  // per query head, at most
  const long long blocks = (long long)G * ((keys_per_head + kWaves * 32 - 1) / (kWaves * 32));
  const int split_tiles = blocks <= kStreamSplitMaxBlocks ? kStreamSplitMinTiles : 4 * kStreamSplitMinTiles;
  const bool split = !(tol > 0.f);
  if (split && blocks <= kStreamSplitMaxBlocks && tiles * rc.kv_group >= kStreamFourMinTiles<D>) A2SF_STREAM(1, 4);
  else if (split && blocks <= 2 * kStreamSplitMaxBlocks && tiles * rc.kv_group >= split_tiles) A2SF_STREAM(1, 2);
  else if (D == 128 && tiles >= kStreamWideMinTiles && blocks >= kStreamWideMinBlocks) A2SF_STREAM((D == 128 ? 2 : 1), 1);
  else A2SF_STREAM(1, 1);
#undef A2SF_STREAM
}

}  // namespace

void launch_attn_bf16(const void* q, const void* k, const void* v, int G, const AttnRect& rc, int d,
                      void* o, float* lse2, hipStream_t st) {
  // a whole prompt (every head's keys are its own rows): the kernels chosen for the prompt phase
  const bool square = !rc.off_heads && !rc.k2 && rc.kv_stride == rc.m;
  if (d == 64) launch_fwd_rect<64>(q, k, v, G, rc, o, lse2, st);
  else if (square) launch_fwd<128>(q, k, v, G, rc.m, o, lse2, st, rc.kv_group, rc.first_row);
  else launch_fwd_rect<128>(q, k, v, G, rc, o, lse2, st);
}

void launch_colscores_bf16(const void* q, const void* k, const float* lse2, int G,
                           const AttnRect& rc, int keys_per_head, int d, float alpha, float* scores,
                           int s_stride, bool accumulate, float decay, hipStream_t st) {
  if (d == 64)
    launch_cols<64>(q, k, lse2, G, rc, keys_per_head, alpha, nullptr, 0.f, scores, s_stride, accumulate, decay, st);
  else
    launch_cols<128>(q, k, lse2, G, rc, keys_per_head, alpha, nullptr, 0.f, scores, s_stride, accumulate, decay, st);
}

// Up to 256 keys always, but for long chains of row blocks of few heads, which the separate kernels split (us per call, separate / one
// kernel, d = 128: 32 heads x 50 rows 15.1 / 12.1, x 250 24.6 / 19.5, 1500 x 250 131 / 116, 32 x 4 queries x 120, 16 row
// blocks, 21.9 / 20.4, but 32 x 6 x 250 at alpha = 0.3, 24, 32.3 / 36.7, chunk of 120 rows of 32 x 4, 16, 32.4 / 33.3; chunk of 50
// rows of 32 heads 21.1 / 17.1).  Up to 512 keys while every workgroup of 16 waves has a compute unit (32 x 260, alpha = 0.5, 22.9 / 19.7,
// chunk of 50 rows behind 300 of 32 heads 29.0 / 25.3, of 200 36.2 / 29.6, but 1500 x 260 164 / 174, 600 chunks 77 / 81), and longer
// prompts only with enough heads to gain from one launch less (500 rows at alpha = 0.3: 200 heads 48 / 46, 32 heads 26.6 / 27.5).
bool scores_select_fits(int G, const AttnRect& rc, int keys_per_head, float alpha) {
  float l2a;
  const int first = first_contributing_row(rc.m, alpha, &l2a);
  const int rows = rc.m - first / kTile * kTile;
  if (keys_per_head > kScoreSelectKeys || rows > kTailTiles * kTile) return false;
  const int chain = (rows + 31) / 32 * rc.kv_group;  // row blocks that a wave goes through
  if (keys_per_head <= 256) return chain <= (rc.k2 ? 8 : 16) || G >= 200;
  return G <= 256 && chain <= 8 && (rc.k2 || keys_per_head <= 320 || G >= 128);
}

void launch_scores_select_bf16(const void* q, const void* k, const void* v, const float* lse2, const AttnRect& rc,
                               int keys_per_head, float alpha, const float* alpha_heads, float decay, float* scores_full,
                               int select, int recent, const a2sf_cache& c, hipStream_t st) {
  const float scale_log2e = 1.4426950408889634f / sqrtf((float)c.d);
  float l2a;
  const int first = first_contributing_row(rc.m, alpha, &l2a);
  const bool chunk = rc.k2 != nullptr;
  const MoveTo to = {(const u32x4_t*)(chunk ? rc.k2 : k), (const u32x4_t*)(chunk ? rc.v2 : v), (u32x4_t*)c.k, (u32x4_t*)c.v,
                     c.scores, c.pos, c.len, c.capacity, lg_row_units(c.d / 8), chunk ? rc.m : 0, nullptr};
#define A2SF_SCORE_SELECT_(D, MOVE, KEYS)                                                             \
  hipLaunchKernelGGL((scores_select_kernel<D, MOVE, KEYS>), dim3(c.G), dim3(kScoreSelectThreads<KEYS>), 0, st, (const bf16_t*)q, \
                     (const bf16_t*)k, lse2, rc, decay, first, l2a, alpha_heads, scale_log2e, scores_full, select, recent, to)
  // Smaller forms leave a compute unit room for more heads: with a room of 256 rows and eight waves whatever the prompt has, many short
  // heads took longer than in two kernels (us per call, two kernels / KEYS = 256 / by size, d = 128: 3000 heads x 34 rows 55.4 / 61.2 / 48.7, 622 x 5
  // queries x 34 48.1 / 52.3 / 44.6, 1345 x 100 50.0 / 50.8 / 45.6, chunks of 30 rows of 1500 heads behind 34 56.8 / 46.2 / 39.7).  For few heads the
  // waves count that move the rows (KEYS = 128 at 32 heads, 20 rows behind 100: 17.2 / 17.9).
#define A2SF_SCORE_SELECT(D, MOVE)                                               \
  do {                                                                           \
    if (keys_per_head <= 64) A2SF_SCORE_SELECT_(D, MOVE, 64);                    \
    else if (keys_per_head <= 128 && c.G > 512) A2SF_SCORE_SELECT_(D, MOVE, 128); \
    else if (keys_per_head <= 256) A2SF_SCORE_SELECT_(D, MOVE, 256);             \
    else A2SF_SCORE_SELECT_(D, MOVE, 512);                                       \
  } while (0)
  if (c.d == 64) {
    if (chunk) A2SF_SCORE_SELECT(64, kInPlace); else A2SF_SCORE_SELECT(64, kGather);
  } else {
    if (chunk) A2SF_SCORE_SELECT(128, kInPlace); else A2SF_SCORE_SELECT(128, kGather);
  }
#undef A2SF_SCORE_SELECT
#undef A2SF_SCORE_SELECT_
}

void launch_prefill_bf16(const void* q, const void* k, const void* v, int G, int n, int d,
                         void* o, float* lse2, hipStream_t st, int first_row) {
  if (d == 64) launch_fwd<64>(q, k, v, G, n, o, lse2, st, 1, first_row);
  else launch_fwd<128>(q, k, v, G, n, o, lse2, st, 1, first_row);
}

int bf16_first_lse_row(int n, float alpha_max) {
  float l2a;
  // the score kernels walk the row tiles from the one that holds the first contributing row
  // on (col_scores_tail_kernel stages them, the other starts its tile loop there; a tile
  // it fetches below that is never used)
  return (first_contributing_row(n, alpha_max, &l2a) / kTile) * kTile;
}

void launch_scores_bf16(const void* q, const void* k, const float* lse2, int G, int n, int d,
                        float alpha, const float* alpha_heads, float tol, float* scores,
                        hipStream_t st) {
  const AttnRect rc{n, n, nullptr};
  if (d == 64)  // (the tolerance is defined for d = 128 only)
    launch_cols<64>(q, k, lse2, G, rc, n, alpha, alpha_heads, 0.f, scores, n, false, 0.f, st);
  else
    launch_cols<128>(q, k, lse2, G, rc, n, alpha, alpha_heads, tol, scores, n, false, 0.f, st);
}

}  // namespace a2sf
