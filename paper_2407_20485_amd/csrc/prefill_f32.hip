// fp32 prompt phase on the fp32 matrix instructions: masked attention rows with their
// log-sum-exp (Section 3.1 Eq.3 of the paper) and the forgotten column scores of Section 3.3
// Eq.5,  S_j = sum_{i>=j} alpha^(n-1-i) * exp(s_ij - lse_i).  Every product and sum is fp32 (the
// instruction multiplies and accumulates in fp32); the probability matrix is recomputed, never
// stored.  The bf16 path lives in prefill_bf16.hip.
//
// Short prompts of few heads go through kernels of plain vector arithmetic instead (below).
//
// Both matrix kernels take the geometry of a2sf_internal.h's AttnRect: m query rows per head against
// keys that lie kv_stride rows apart from head to head; row i sees keys 0 .. off + i, where
// off (per head, or 0) is the number of older tokens in front of the rows' own.  The prompt
// phase is the square case (off = 0, kv_stride = m); a chunk of a prompt runs against the
// head's cache (off = tokens cached before the chunk).
//
// Operand layouts of v_mfma_f32_32x32x2_f32: lane (x = lane % 32, h = lane / 32) brings A[x][k = h]
// and B[k = h][x]; accumulator register i of the lane is row 8 (i/4) + 4 h + i % 4, column x.
// Both kernels form the transposed logit tile (keys = rows, queries = columns), so a lane owns
// one query, and register i of the tile is at once the B operand of the i-th step of
// O^T = V^T P^T (its two halves bring the keys 8 (i/4) + i % 4 and + 4).  The order in which a
// sum over d runs is free: lane half h takes the elements 8c + 4h .. + 3 in the steps 4c .. 4c+3,
// so operands come as 16-byte pieces.
//
// One matrix op takes 64 cycles of its pipe for two operand floats per lane, so tiles need not
// be shared: a wave fetches its own 32-row tiles straight into its own LDS strip
// (global_load_lds) and meets the other waves of its workgroup only at the end.  The four waves of a
// workgroup share 32 query rows (attention) or 32 keys (scores) and take every fourth tile, which keeps
// the chip full from a few hundred rows on and the longest row's chain short.
// 32 heads x 1000 rows x 128: attention 101 us (8.2 GFLOP = 81 TFLOP/s of the 154 that a large fp32
// matrix product reaches), scores 23 us (window of 93 rows; vector form: 219).
#include <math.h>

#include "a2sf_dev.h"
#include "a2sf_internal.h"

namespace a2sf {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) char lds_char;

constexpr int kRows = 32;  // query rows (attention) / keys (scores) per workgroup, and rows of a tile

__device__ __forceinline__ f32x16 mfma_f32(float a, float b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 lds_read4(const lds_char* p) {
  return *reinterpret_cast<const __attribute__((address_space(3))) f32x4*>(p);
}
__device__ __forceinline__ float lds_read1(const lds_char* p) {
  return *reinterpret_cast<const __attribute__((address_space(3))) float*>(p);
}

// 16-byte chunks of a tile row are stored at chunk ^ swizzle(row).  Tiles read 16 rows x one
// chunk column per 16 lanes (K, Q): the row's low bits send them to 16 different bank groups.
// V is read as 32 consecutive floats of a key per half of the wave, the halves 4 keys apart: they
// get different 32-float groups.
template <bool V_LAYOUT>
__device__ __forceinline__ int tile_swizzle(int row) { return V_LAYOUT ? ((row >> 2) & 1) * 8 : (row & 15); }

// Rows row0 .. row0 + 31 of Mg (clamped to n rows) into this wave's LDS tile: D / 8 loads.
template <int D, bool V_LAYOUT>
__device__ __forceinline__ void fetch_tile(const float* __restrict__ Mg, int row0, int n, lds_char* tile) {
  constexpr int CPR = D / 4, RPL = 64 / CPR;  // chunks per row, rows per load
  const int lane = threadIdx.x & 63;
  const float* base = Mg + (size_t)row0 * D;
  const int most = n - 1 - row0;
#pragma unroll
  for (int u = 0; u < kRows / RPL; ++u) {
    const int lrow = u * RPL + lane / CPR, pc = lane % CPR;
    const int c = pc ^ tile_swizzle<V_LAYOUT>(lrow);
    dma16(base, (uint32_t)(min(lrow, most) * D * 4 + c * 16), (uint32_t)(size_t)(tile + u * 1024));
  }
}

// The maximum that a row's exponents are taken against is that of the logits as they come from the products, before
// they are scaled, so that the largest one's exponent is exactly 0 however large it is (s * scale rounded and s * scale in
// an fma differ by more than an exponent's range from 2^31 on).  It starts here and not at -inf, which must not be
// subtracted from a masked logit.
constexpr float kLowest = -3.402823466e38f;

// A matrix op multiplies a masked key's probability, 0, with its V row, and 0 times an infinity is not 0.
// So the tiles that the mask cuts are looked over (D / 8 LDS reads of a lane beside the 4 D of the products) and their
// infinities and NaN set to 0; add_nonfinite gives them to the rows that see them at the end.
template <int D>
__device__ __forceinline__ bool clear_nonfinite(lds_char* tile) {
  lds_char* const mine = tile + (threadIdx.x & 63) * 16;
  float zeros = 0.f;  // a NaN if some x is not finite
#pragma unroll 4
  for (int u = 0; u < D / 8; ++u) {
    const f32x4 x = lds_read4(mine + u * 1024);
    zeros = fmaf(x[0], 0.f, fmaf(x[1], 0.f, fmaf(x[2], 0.f, fmaf(x[3], 0.f, zeros))));
  }
  if (!__any(zeros != 0.f)) return false;
#pragma unroll 1
  for (int u = 0; u < D / 8; ++u) {
    f32x4 x = lds_read4(mine + u * 1024);
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = x[e] * 0.f == 0.f ? x[e] : 0.f;
    *reinterpret_cast<__attribute__((address_space(3))) f32x4*>(mine + u * 1024) = x;
  }
  return true;
}
// The terms p v of the keys [key0, last key of the row] whose v is not finite, onto the rows that a workgroup has
// stored (such a sum is an infinity or NaN: adding a term again, or p's own rounding, does not change it).
template <int D>
__device__ __forceinline__ void add_nonfinite(const float* Qg, const float* Kg, const float* Vg, const float* lse2, float* Og,
                                           int row0, int n, int off, int key0, float scale_log2e) {
  for (int e = threadIdx.x; e < kRows * D; e += kThreads) {
    const int r = row0 + e / D, c = e % D;
    if (r >= n) break;
    float x = Og[(size_t)r * D + c];
    for (int j = key0; j <= off + r; ++j) {
      const float v = Vg[(size_t)j * D + c];
      if (v * 0.f == 0.f) continue;
      float s = 0.f;
      for (int i = 0; i < D; ++i) s = fmaf(Qg[(size_t)r * D + i], Kg[(size_t)j * D + i], s);
      x += exp2f(fmaf(s, scale_log2e, -lse2[r])) * v;
    }
    Og[(size_t)r * D + c] = x;
  }
}

// One workgroup per 32 query rows; wave w takes the key tiles w, w + 4, ...  A wave's strip holds
// the K tile until its logits are formed, then the V tile: the wave waits for each, and the
// second wave of the SIMD fills the gaps (two strips per wave, with the next tile fetched half a tile ahead,
// leave room for one wave per SIMD only: 126 us instead of 117 at 32 heads x 1000 rows x 128 in the old launch order;
// quarters of a tile fetched as the quarters before them are used up: no difference; a workgroup of
// vector arithmetic per row, as this kernel used to be: 2187).
template <int D, bool WITH_O>
__global__ __launch_bounds__(kThreads, D == 64 ? 3 : 2) void attn_f32_kernel(
    const float* __restrict__ Q, const float* __restrict__ K, const float* __restrict__ V,
    AttnRect rc, int GQ, int nqb, float* __restrict__ O, float* __restrict__ LSE2, float scale_log2e) {
  constexpr int C8 = D / 8, DB = D / 32, kTileBytes = kRows * D * 4;
  __shared__ __attribute__((aligned(1024))) char smem[kWaves * kTileBytes];
  __shared__ float m_s[kWaves][kRows], l_s[kWaves][kRows];
  __shared__ bool odd_s[kWaves];

  int g, rank;
  if (!ordered_item(GQ, nqb, g, rank)) return;
  const int qb = rc.first_row / kRows + nqb - 1 - rank;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, h = lane >> 5;
  const int n = rc.m, row0 = qb * kRows;
  const int gk = g / rc.kv_group;  // the K/V head this query head reads
  const int off = rc.off_heads ? rc.off_heads[gk] : 0;
  if (off < 0) {  // a head the caller's precondition excludes: its rows are flagged
    if (WITH_O)
      for (int e = tid; e < min(kRows, n - row0) * D; e += kThreads)
        O[((size_t)g * n + row0) * D + e] = __int_as_float(0x7FC00000);
    return;
  }
  const int nk = off + n;
  const float* Kg = K + (size_t)gk * rc.kv_stride * D;
  const float* Vg = V + (size_t)gk * rc.kv_stride * D;
  lds_char* const strip = (lds_char*)smem + wave * kTileBytes;

  const int last_key = off + min(n, row0 + kRows) - 1;
  const int ntiles = last_key / kRows + 1;
  if (wave < ntiles) fetch_tile<D, false>(Kg, wave * kRows, nk, strip);
  // Q (B operand): lane (query l32, half h) holds the elements 8c + 4h .. + 3
  f32x4 qf[C8];
  {
    const float* qr = Q + ((size_t)g * n + min(row0 + l32, n - 1)) * D + 4 * h;
#pragma unroll
    for (int c = 0; c < C8; ++c) qf[c] = *reinterpret_cast<const f32x4*>(qr + 8 * c);
  }
#pragma unroll
  for (int c = 0; c < C8; ++c) asm volatile("" : "+v"(qf[c]));  // waited for here, not in every round of the loop
  int koff[C8 < 8 ? C8 : 8];  // chunk 2c + h of row l32: the swizzle reaches the low four chunk bits
#pragma unroll
  for (int c = 0; c < 8 && c < C8; ++c) koff[c] = l32 * D * 4 + (((2 * c + h) ^ tile_swizzle<false>(l32)) << 4);
  const int voff[2] = {4 * h * D * 4 + l32 * 4 + h * 128, 4 * h * D * 4 + l32 * 4 + (1 - h) * 128};

  f32x16 oacc[WITH_O ? DB : 1];
#pragma unroll
  for (int db = 0; db < (WITH_O ? DB : 1); ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) oacc[db][i] = 0.f;
  float m = kLowest, l = 0.f;
  bool odd = false;  // a V row of a masked tile holds an infinity or a NaN
  const int newest = off + row0 + l32;  // newest key this lane's row sees

  for (int t = wave; t < ntiles; t += kWaves) {
    const int key0 = t * kRows, next = min(t + kWaves, ntiles - 1) * kRows;
    wait_vm<0>();  // K tile t
    f32x16 s, s2;  // two sums: no matrix op waits for the one before it, and each rounds half as often
#pragma unroll
    for (int i = 0; i < 16; ++i) s[i] = s2[i] = 0.f;
#pragma unroll
    for (int c = 0; c < C8; ++c) {
      const f32x4 kf = lds_read4(strip + koff[c & 7] + (c >> 3) * 256);
#pragma unroll
      for (int j = 0; j < 4; j += 2) {
        s = mfma_f32(kf[j], qf[c][j], s);
        s2 = mfma_f32(kf[j + 1], qf[c][j + 1], s2);
      }
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) s[i] += s2[i];
    wait_lds();
    if (WITH_O) fetch_tile<D, true>(Vg, key0, nk, strip);
    else fetch_tile<D, false>(Kg, next, nk, strip);
    const bool masked = key0 + kRows - 1 > off + row0;  // the tile reaches past the block's first row
    if (masked) {
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (key0 + 8 * (i >> 2) + 4 * h + (i & 3) > newest) s[i] = -INFINITY;
    }
    float mx = s[0];
#pragma unroll
    for (int i = 1; i < 16; ++i) mx = fmaxf(mx, s[i]);
    mx = across_rows(mx, OpMax(), false, true);
    const float m_new = fmaxf(m, mx);
    if (__any(m_new > m)) {
      const float corr = exp2f((m - m_new) * scale_log2e);
      l *= corr;
      if (WITH_O) {
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
          for (int i = 0; i < 16; ++i) oacc[db][i] *= corr;
      }
      m = m_new;
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      s[i] = __builtin_amdgcn_exp2f((s[i] - m) * scale_log2e);
      l += s[i];
    }
    if constexpr (WITH_O) {
      wait_vm<0>();  // V tile t
      if (masked && clear_nonfinite<D>(strip)) {
        odd = true;
        wait_lds();
      }
#pragma unroll
      for (int i = 0; i < 16; ++i) {
#pragma unroll
        for (int db = 0; db < DB; ++db) {
          const float vf = lds_read1(strip + voff[db & 1] + (db >> 1) * 256 + (8 * (i >> 2) + (i & 3)) * D * 4);
          oacc[db] = mfma_f32(vf, s[i], oacc[db]);
        }
      }
      wait_lds();
      fetch_tile<D, false>(Kg, next, nk, strip);
    }
  }
  wait_vm<0>();  // the strip is reused below

  // ---- the four waves' parts of the 32 rows
  l = across_rows(l, OpAdd(), false, true);
  if (h == 0) { m_s[wave][l32] = m; l_s[wave][l32] = l; }
  if (WITH_O && lane == 0) odd_s[wave] = odd;
  __syncthreads();
  float mall = m_s[0][l32];
#pragma unroll
  for (int w = 1; w < kWaves; ++w) mall = fmaxf(mall, m_s[w][l32]);
  float lall = 0.f;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) lall += l_s[w][l32] * exp2f((m_s[w][l32] - mall) * scale_log2e);
  if (wave == 0 && h == 0 && row0 + l32 < n)
    LSE2[(size_t)g * n + row0 + l32] = fmaf(mall, scale_log2e, log2f(lall));
  if constexpr (WITH_O) {
    const float f = exp2f((m - mall) * scale_log2e) / lall;
    // the strip now takes the wave's outputs, [query][d], chunks swizzled as in a tile
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4) {
        const f32x4 w = {oacc[db][4 * i4] * f, oacc[db][4 * i4 + 1] * f, oacc[db][4 * i4 + 2] * f,
                         oacc[db][4 * i4 + 3] * f};
        const int chunk = 8 * db + 2 * i4 + h;
        *reinterpret_cast<__attribute__((address_space(3))) f32x4*>(
            strip + l32 * D * 4 + ((chunk ^ tile_swizzle<false>(l32)) << 4)) = w;
      }
    __syncthreads();
    constexpr int CPR = D / 4;
    for (int u = tid; u < kRows * CPR; u += kThreads) {
      const int r = u / CPR, c = u % CPR;
      if (row0 + r >= n) break;
      const lds_char* p = (const lds_char*)smem + r * D * 4 + ((c ^ tile_swizzle<false>(r)) << 4);
      const f32x4 a = (lds_read4(p) + lds_read4(p + kTileBytes)) +
                      (lds_read4(p + 2 * kTileBytes) + lds_read4(p + 3 * kTileBytes));
      *reinterpret_cast<f32x4*>(O + ((size_t)g * n + row0 + r) * D + c * 4) = a;
    }
    if (odd_s[0] || odd_s[1] || odd_s[2] || odd_s[3]) {
      __syncthreads();
      add_nonfinite<D>(Q + (size_t)g * n * D, Kg, Vg, LSE2 + (size_t)g * n, O + (size_t)g * n * D, row0, n, off,
                       (off + row0) / kRows * kRows, scale_log2e);
    }
  }
}

// One workgroup per 32 keys, whose K rows stay in registers; wave w takes every fourth tile of 32
// query rows of the head's kv_group query heads.  `accumulate`: the result is added to `decay`
// times what scores[] holds (a chunk: the cached tokens' older scores, decayed by alpha^m);
// otherwise it replaces it.
template <int D>
__global__ __launch_bounds__(kThreads, 2) void scores_f32_kernel(
    const float* __restrict__ Q, const float* __restrict__ K, const float* __restrict__ LSE2,
    AttnRect rc, int G, int ncb, int first_row, float log2_alpha, const float* __restrict__ alpha_heads,
    float* __restrict__ scores, int s_stride, bool accumulate, float decay, float scale_log2e) {
  constexpr int C8 = D / 8, kTileBytes = kRows * D * 4;
  __shared__ __attribute__((aligned(1024))) char smem[kWaves * kTileBytes];
  __shared__ float part[kWaves][kRows];
  int g, rank;
  if (!ordered_item(G, ncb, g, rank)) return;
  const int c0 = rank * kRows;  // the oldest keys have the most rows
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, h = lane >> 5;
  const int n = rc.m;
  const int off = rc.off_heads ? rc.off_heads[g] : 0;
  const int nk = off + n;
  if (off < 0 || c0 >= nk) return;
  head_window(alpha_heads, g, n, first_row, log2_alpha);
  const float* Qg = Q + (size_t)g * rc.kv_group * n * D;  // the group's rows lie one head after the other
  const float* lg = LSE2 + (size_t)g * rc.kv_group * n;
  lds_char* const qt = (lds_char*)smem + wave * kTileBytes;

  const int t0 = max(max(c0 - off, first_row), 0) / kRows;  // first row tile that counts
  const int nt = (n + kRows - 1) / kRows - t0;              // tiles per query head
  const int work = nt * rc.kv_group;
  auto fetch = [&](int f) {
    const int hq = f / nt, t = t0 + f % nt;
    fetch_tile<D, false>(Qg + (size_t)hq * n * D, t * kRows, n, qt);
  };
  if (wave < work) fetch(wave);
  f32x4 kf[C8];  // A operand: lane (key l32, half h) holds the elements 8c + 4h .. + 3
  {
    const float* kr = K + ((size_t)g * rc.kv_stride + min(c0 + l32, nk - 1)) * D + 4 * h;
#pragma unroll
    for (int c = 0; c < C8; ++c) kf[c] = *reinterpret_cast<const f32x4*>(kr + 8 * c);
  }
#pragma unroll
  for (int c = 0; c < C8; ++c) asm volatile("" : "+v"(kf[c]));  // waited for here, not in every round of the loop
  int qoff[C8 < 8 ? C8 : 8];
#pragma unroll
  for (int c = 0; c < 8 && c < C8; ++c) qoff[c] = l32 * D * 4 + (((2 * c + h) ^ tile_swizzle<false>(l32)) << 4);
  float acc[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = 0.f;

  for (int f = wave; f < work; f += kWaves) {
    const int hq = f / nt, r = (t0 + f % nt) * kRows + l32;
    float lse = lg[(size_t)hq * n + min(r, n - 1)];
    asm volatile("" : "+v"(lse));  // with the tile: everything has arrived
    wait_vm<0>();
    f32x16 s, s2;
#pragma unroll
    for (int i = 0; i < 16; ++i) s[i] = s2[i] = 0.f;
#pragma unroll
    for (int c = 0; c < C8; ++c) {
      const f32x4 qf = lds_read4(qt + qoff[c & 7] + (c >> 3) * 256);
#pragma unroll
      for (int j = 0; j < 4; j += 2) {
        s = mfma_f32(kf[c][j], qf[j], s);
        s2 = mfma_f32(kf[c][j + 1], qf[j + 1], s2);
      }
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) s[i] += s2[i];
    wait_lds();
    if (f + kWaves < work) fetch(f + kWaves);
    // exponent offset of row r: lse_r - (n-1-r) log2(alpha); rows past the end, and rows whose
    // weight is exactly 0 in fp32 (before first_row), add nothing
    const bool counts = r < n && r >= first_row;
    const float w = (float)(n - 1 - r) * log2_alpha;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const float p = exp2f(fmaf(s[i], scale_log2e, -lse) + w);
      const int key = c0 + 8 * (i >> 2) + 4 * h + (i & 3);
      acc[i] += counts && key <= off + r ? p : 0.f;
    }
  }
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    acc[i] = group_sum<32>(acc[i]);  // over the 32 rows held by the lanes of one half
    if (l32 == 0) part[wave][8 * (i >> 2) + 4 * h + (i & 3)] = acc[i];
  }
  __syncthreads();
  if (tid < kRows && c0 + tid < nk) {
    const float sum = (part[0][tid] + part[1][tid]) + (part[2][tid] + part[3][tid]);
    float* out = scores + (size_t)g * s_stride + c0 + tid;
    *out = accumulate ? fmaf(decay, *out, sum) : sum;
  }
}

// ---- short prompts -------------------------------------------------------------------------
// A matrix op of 64 cycles per two elements makes a tile of 32 rows a chain of 8000 cycles and more, whatever the
// prompt has of it.  A short prompt of few heads is done sooner by plain arithmetic: a workgroup per attention row, then one
// per key (square geometry only).
constexpr int kShortRows = 512;  // of a prompt, at most

template <int D>
__device__ __forceinline__ float dot_row(const float* __restrict__ a, const float* __restrict__ b) {
  float acc = 0.f;
#pragma unroll
  for (int c = 0; c < D; c += 4) {
    const float4 x = *reinterpret_cast<const float4*>(a + c);
    const float4 y = *reinterpret_cast<const float4*>(b + c);
    acc = fmaf(x.x, y.x, acc); acc = fmaf(x.y, y.y, acc);
    acc = fmaf(x.z, y.z, acc); acc = fmaf(x.w, y.w, acc);
  }
  return acc;
}

template <int D>
__global__ __launch_bounds__(kThreads) void attn_rows_f32_kernel(
    const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v,
    AttnRect rc, float* __restrict__ o, float* __restrict__ lse2, float scale_log2e) {
  __shared__ float z[kShortRows];
  __shared__ float part[kThreads / D][D];
  __shared__ float red[8];
  const int n = rc.m, rows = n - rc.first_row;
  const int g = blockIdx.x / rows, i = rc.first_row + blockIdx.x % rows, tid = threadIdx.x;
  const int gk = g / rc.kv_group;  // the K/V head this query head reads
  const float* qi = q + ((size_t)g * n + i) * D;
  const float* kg = k + (size_t)gk * rc.kv_stride * D;
  const float* vg = v + (size_t)gk * rc.kv_stride * D;
  constexpr int PARTS = kThreads / D;
  const int c = tid % D, part_id = tid / D;

  float m = -INFINITY, l = 0.f, acc = 0.f;
  for (int j = tid; j <= i; j += kThreads) {
    z[j] = dot_row<D>(qi, kg + (size_t)j * D) * scale_log2e;
    m = fmaxf(m, z[j]);
  }
  m = block_max(m, red);
  for (int j = tid; j <= i; j += kThreads) {
    z[j] = exp2f(z[j] - m);
    l += z[j];
  }
  l = block_sum(l, red);
  if (o) {
    for (int j = part_id; j <= i; j += PARTS) acc = fmaf(z[j], vg[(size_t)j * D + c], acc);
    part[part_id][c] = acc;
    __syncthreads();
    if (tid < D) {
      float t = 0.f;
#pragma unroll
      for (int p = 0; p < PARTS; ++p) t += part[p][tid];
      o[((size_t)g * n + i) * D + tid] = t / l;
    }
  }
  if (tid == 0) lse2[(size_t)g * n + i] = m + log2f(l);
}

// Column scores, one workgroup per key.
template <int D>
__global__ __launch_bounds__(kThreads) void scores_rows_f32_kernel(
    const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ lse2,
    AttnRect rc, int first_row, float log2_alpha, const float* __restrict__ alpha_heads,
    float* __restrict__ scores, int s_stride, float scale_log2e) {
  __shared__ float red[8];
  const int n = rc.m;
  const int g = blockIdx.x / n, j = blockIdx.x % n, tid = threadIdx.x;
  head_window(alpha_heads, g, n, first_row, log2_alpha);
  const float* kj = k + ((size_t)g * rc.kv_stride + j) * D;
  float sum = 0.f;
  for (int hq = 0; hq < rc.kv_group; ++hq) {  // the query heads that share this K/V head
    const float* qg = q + ((size_t)g * rc.kv_group + hq) * n * D;
    const float* lg = lse2 + ((size_t)g * rc.kv_group + hq) * n;
    for (int i = max(j, first_row) + tid; i < n; i += kThreads) {
      const float s = dot_row<D>(qg + (size_t)i * D, kj) * scale_log2e;
      sum += exp2f(s - lg[i] + (float)(n - 1 - i) * log2_alpha);
    }
  }
  sum = block_sum(sum, red);
  if (tid == 0) scores[(size_t)g * s_stride + j] = sum;
}

}  // namespace

int first_contributing_row(int n, float alpha, float* log2_alpha) {
  if (alpha <= 0.f) { *log2_alpha = 0.f; return n - 1; }
  if (alpha >= 1.f) { *log2_alpha = 0.f; return 0; }
  const float l2 = log2f(alpha);  // < 0
  *log2_alpha = l2;
  // weight 2^((n-1-i)*l2) <= 2^-160 rounds to 0 in fp32 whatever the probability (<= 1)
  const double rows = 160.0 / (double)(-l2);
  if (rows >= (double)n) return 0;
  const int w = (int)rows + 1;
  return n - w < 0 ? 0 : n - w;
}

// The kernels by rows cost G n workgroups of up to n keys, those by tiles a chain of n / 128: they meet where G n^1.5 is
// about constant (us, attention and scores, rows / tiles: d = 128, 1 head x 200 21 / 23, x 300 30 / 30, 8 x 64 13 / 19, 8
// x 130 28 / 23, 40 x 20 13 / 18, 40 x 48 26 / 20, 300 x 5 14 / 19, 300 x 12 32 / 20; d = 64, 1 x 420 23 / 26, 8 x 96 11 /
// 14, 40 x 32 9 / 14, 40 x 64 18 / 14, 300 x 5 8 / 14, 300 x 20 23 / 15).
static bool short_prompt(int G, const AttnRect& rc, int d) {
  const double rows = (double)G * rc.kv_group * rc.m;
  return !rc.off_heads && rc.m <= kShortRows && rows * rows * rc.m <= (d == 64 ? 90e6 : 27e6);
}

void launch_attn_f32(const float* q, const float* k, const float* v, int G, const AttnRect& rc,
                     int d, float* o, float* lse2, hipStream_t st) {
  const float scale_log2e = 1.4426950408889634f / sqrtf((float)d);
  const int GQ = G * rc.kv_group;
  if (short_prompt(G, rc, d)) {
    const dim3 rows((unsigned)GQ * (unsigned)(rc.m - rc.first_row));
    if (d == 64) hipLaunchKernelGGL(attn_rows_f32_kernel<64>, rows, dim3(kThreads), 0, st, q, k, v, rc, o, lse2, scale_log2e);
    else hipLaunchKernelGGL(attn_rows_f32_kernel<128>, rows, dim3(kThreads), 0, st, q, k, v, rc, o, lse2, scale_log2e);
    return;
  }
  const int nqb = (rc.m + kRows - 1) / kRows - rc.first_row / kRows;  // row blocks to compute
  const unsigned grid = ordered_grid(GQ, nqb);
#define A2SF_ATTN_F32(D, WO)                                                                          \
  hipLaunchKernelGGL((attn_f32_kernel<D, WO>), dim3(grid), dim3(kThreads), 0, st, q, k, v, rc, GQ, nqb, o, \
                     lse2, scale_log2e)
  if (d == 64) {
    if (o) A2SF_ATTN_F32(64, true); else A2SF_ATTN_F32(64, false);
  } else {
    if (o) A2SF_ATTN_F32(128, true); else A2SF_ATTN_F32(128, false);
  }
#undef A2SF_ATTN_F32
}

void launch_colscores_f32(const float* q, const float* k, const float* lse2, int G,
                          const AttnRect& rc, int keys_per_head, int d, float alpha,
                          const float* alpha_heads, float* scores, int s_stride, bool accumulate,
                          float decay, hipStream_t st) {
  const float scale_log2e = 1.4426950408889634f / sqrtf((float)d);
  float l2a;
  const int first = first_contributing_row(rc.m, alpha, &l2a);
  if (short_prompt(G, rc, d)) {
    const dim3 keys((unsigned)G * (unsigned)rc.m);
    if (d == 64)
      hipLaunchKernelGGL(scores_rows_f32_kernel<64>, keys, dim3(kThreads), 0, st, q, k, lse2, rc, first, l2a, alpha_heads,
                         scores, s_stride, scale_log2e);
    else
      hipLaunchKernelGGL(scores_rows_f32_kernel<128>, keys, dim3(kThreads), 0, st, q, k, lse2, rc, first, l2a, alpha_heads,
                         scores, s_stride, scale_log2e);
    return;
  }
  const int ncb = (keys_per_head + kRows - 1) / kRows;
  const unsigned grid = ordered_grid(G, ncb);
  if (d == 64)
    hipLaunchKernelGGL(scores_f32_kernel<64>, dim3(grid), dim3(kThreads), 0, st, q, k, lse2, rc, G, ncb, first,
                       l2a, alpha_heads, scores, s_stride, accumulate, decay, scale_log2e);
  else
    hipLaunchKernelGGL(scores_f32_kernel<128>, dim3(grid), dim3(kThreads), 0, st, q, k, lse2, rc, G, ncb, first,
                       l2a, alpha_heads, scores, s_stride, accumulate, decay, scale_log2e);
}

void launch_prefill_f32(const float* q, const float* k, const float* v, int G, int n, int d,
                        float* o, float* lse2, hipStream_t st, int first_row) {
  AttnRect rc{n, n, nullptr};
  rc.first_row = o ? 0 : first_row;
  launch_attn_f32(q, k, v, G, rc, d, o, lse2, st);
}

int f32_first_lse_row(int n, float alpha_max) {
  float l2a;
  return first_contributing_row(n, alpha_max, &l2a);
}

void launch_scores_f32(const float* q, const float* k, const float* lse2, int G, int n, int d,
                       float alpha, const float* alpha_heads, float* scores, hipStream_t st) {
  launch_colscores_f32(q, k, lse2, G, AttnRect{n, n, nullptr}, n, d, alpha, alpha_heads, scores, n,
                       false, 0.f, st);
}

}  // namespace a2sf
