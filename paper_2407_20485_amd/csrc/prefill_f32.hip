// fp32 prompt phase on the matrix cores, to the precision of fp32: masked attention rows with their
// log-sum-exp (Section 3.1 Eq.3 of the paper) and the forgotten column scores of Section 3.3
// Eq.5,  S_j = sum_{i>=j} alpha^(n-1-i) * exp(s_ij - lse_i).  The probability matrix is recomputed, never
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
// Products run on v_mfma_f32_32x32x16_bf16, which does sixteen times the multiplications of the fp32 instruction per
// cycle: every fp32 operand is split into three bf16 parts, high + middle + low, which together are the number itself (the
// splitting of Henry, Tang and Heinecke, "Leveraging the bfloat16 Artificial Intelligence Datatype For
// Higher-Precision Computations", 2019), and six of the nine products of parts are summed in fp32 (the instruction
// multiplies exactly).  High and middle parts are rounded to nearest, so a middle part is at most 2^-8 of its number and a low
// part 2^-17; what is dropped, middle x low twice and low x low, is at most 2^-24 of the product, with no sign in
// common: never more than one rounding of fp32, and nothing that adds up (parts that are cut off instead drop up to 2^-21,
// always towards zero).  The corrections of a logit are summed apart from its high parts; a tile's share of an output is summed
// on its own.  Relative error against 64 bits, of sums of 128 products, on a model of the arithmetic: normal values 5.7e-8 (fp32
// multiply-adds 1.5e-7, cut parts 8.2e-8), one nonzero product 2.6e-8 (2.5e-8, 6.4e-8), two 2.7e-8 (3.7e-8, 6.6e-8).
//
// Not every number has its parts in the range of bf16: an infinity, a NaN and what rounds to one (above 2^127.99) have none, and the
// parts of a number below 2^-110 end at 2^-133, where a subnormal bf16 does.  What that costs is 2^-134 times the other operand, so it
// matters where the other one is large, or the result small: a workgroup that has rows with numbers below 2^-110 or above
// 2^100 (of Q in the attention, of K in the scores), or outputs below 2^-106 or not finite, does its block once more with
// such logits and products in plain fp32 arithmetic, or in parts of larger multiples (`careful` below).  What is left is 2^-20
// of a logit's unit and 2^-28 of an output; probabilities below 2^-110 of their row's largest are off by up to 2^-134, where the
// exponential itself ends at 2^-126.
//
// Operand layouts: lane (x = lane % 32, h = lane / 32) brings A[x][k] and B[k][x] for the eight k of its half;
// accumulator register i of the lane is row 8 (i/4) + 4 h + i % 4, column x.  Both kernels form the transposed logit
// tile (keys = rows, queries = columns), so a lane owns one query, and the registers 8j .. 8j+7 of the tile
// are at once the B operand of step j of O^T = V^T P^T (a half brings the keys 16j + 4h .. +3 and 16j + 8 + 4h .. +3).
// A sum over d runs in steps of 16 elements, eight to a half, so operands come as 16-byte pieces.
//
// Waves fetch 32-row tiles straight into LDS (global_load_lds) and cut what they read from there.  The waves of
// a workgroup share 32 or 64 query rows (attention) or 32 keys (scores) and take the tiles in turn, which keeps
// the chip full from a few hundred rows on and the longest row's chain short; they add up at the end.
// Scores of 32 heads x 1000 rows (window of 93 rows): 22 us.
#include <math.h>

#include <type_traits>

#include "a2sf_dev.h"
#include "a2sf_internal.h"

namespace a2sf {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) char lds_char;

constexpr int kRows = 32;  // query rows (attention) / keys (scores) per workgroup, and rows of a tile

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
__device__ __forceinline__ f32x16 mfma_bf16(const uint4& a, const uint4& b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
// Eight numbers as three bf16 operands whose sum they are: 24 bits in three times eight, high and middle rounded to nearest, so that
// every difference is exact and the last one has no more than eight bits.
struct Parts {
  uint4 high, middle, low;
};
__device__ __forceinline__ Parts split(const float (&x)[8]) {
  uint32_t hi[4], mi[4], lo[4];
  const auto upper = [](float a, float b) { return __builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x07060302u); };
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    float h[2], r[2], m[2], rr[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      // (a pair with a zero below is the rounded number in fp32: a pair of two has to be taken apart again by instructions that wait for each other)
      h[e] = __uint_as_float(pack_bf16(0.f, x[2 * i + e]));
      r[e] = x[2 * i + e] - h[e];
      m[e] = __uint_as_float(pack_bf16(0.f, r[e]));
      rr[e] = r[e] - m[e];
    }
    hi[i] = upper(h[0], h[1]);
    mi[i] = upper(m[0], m[1]);
    lo[i] = upper(rr[0], rr[1]);
  }
  return {make_uint4(hi[0], hi[1], hi[2], hi[3]), make_uint4(mi[0], mi[1], mi[2], mi[3]), make_uint4(lo[0], lo[1], lo[2], lo[3])};
}
__device__ __forceinline__ Parts split(const f32x4& a, const f32x4& b) {
  const float x[8] = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
  return split(x);
}
// The number that element e of eight was split from.
__device__ __forceinline__ float joined(const Parts& p, int e) {
  const auto part = [&](const uint4& w) {
    const uint32_t pair = (e >> 1) == 0 ? w.x : (e >> 1) == 1 ? w.y : (e >> 1) == 2 ? w.z : w.w;
    return __uint_as_float(e & 1 ? pair & 0xFFFF0000u : pair << 16);
  };
  return (part(p.high) + part(p.middle)) + part(p.low);
}
// sum += the product of the high parts, rest += the five next largest ones
__device__ __forceinline__ void multiply(const Parts& a, const Parts& b, f32x16& sum, f32x16& rest) {
  rest = mfma_bf16(a.low, b.high, rest);
  sum = mfma_bf16(a.high, b.high, sum);
  rest = mfma_bf16(a.high, b.low, rest);
  rest = mfma_bf16(a.middle, b.middle, rest);
  rest = mfma_bf16(a.middle, b.high, rest);
  rest = mfma_bf16(a.high, b.middle, rest);
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

// Rows row0 .. row0 + 31 of Mg (clamped to n rows) into an LDS tile, the loads first, first + step, ... of its D / 8.
// In a tile that lies inside the matrix a load's lane offsets differ from the first one's by an exclusive or (the
// rows of a load have the bits below its own first row) and by whole loads, which the scalar base takes.
template <int D, bool V_LAYOUT>
__device__ __forceinline__ void fetch_tile(const float* __restrict__ Mg, int row0, int n, lds_char* tile, int first = 0,
                                           int step = 1) {
  constexpr int CPR = D / 4, RPL = 64 / CPR;  // chunks per row, rows per load
  int lane = threadIdx.x & 63;
  const float* base = Mg + (size_t)row0 * D;
  const int most = n - 1 - row0;
  if (most >= kRows - 1) {
    uint32_t lane0 = (uint32_t)((lane % CPR ^ tile_swizzle<V_LAYOUT>(lane / CPR)) * 16 + lane / CPR * D * 4);
    asm volatile("" : "+v"(lane0));  // (the others are formed here: kept over a kernel's loop they are more registers than it has)
#pragma unroll
    for (int u = 0; u < kRows / RPL; ++u)
      if (u % step == first)
        dma16(base + u * RPL * D, lane0 ^ (uint32_t)(tile_swizzle<V_LAYOUT>(u * RPL) * 16), (uint32_t)(size_t)(tile + u * 1024));
  } else {
    asm volatile("" : "+v"(lane));
#pragma unroll
    for (int u = 0; u < kRows / RPL; ++u) {
      const int lrow = u * RPL + lane / CPR, pc = lane % CPR;
      const int c = pc ^ tile_swizzle<V_LAYOUT>(lrow);
      if (u % step == first) dma16(base, (uint32_t)(min(lrow, most) * D * 4 + c * 16), (uint32_t)(size_t)(tile + u * 1024));
    }
  }
}

// The maximum that a row's exponents are taken against is that of the logits as they come from the products, before
// they are scaled, so that the largest one's exponent is exactly 0 however large it is (s * scale rounded and s * scale in
// an fma differ by more than an exponent's range from 2^31 on).  It starts here and not at -inf, which must not be
// subtracted from a masked logit.
constexpr float kLowest = -3.402823466e38f;

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

// Which operands the parts cannot stand for (see the top of the file).
constexpr float kSmallestSplit = 0x1p-110f, kLargestSplit = 0x1p127f, kLargestRow = 0x1p100f, kSmallestSum = 0x1p-106f, kLargest = 3.402823466e38f;
__device__ __forceinline__ bool has_parts(float x) { return x == 0.f || (fabsf(x) >= kSmallestSplit && fabsf(x) <= kLargestSplit); }
__device__ __forceinline__ bool finite(float x) { return fabsf(x) < INFINITY; }
// The extremes of numbers, and where a zero may be the least of them, whether another one is too small.
struct Extremes {
  float most = 0.f, least = INFINITY;
  __device__ __forceinline__ void see(const f32x4& x) {
    most = __builtin_elementwise_maximum(__builtin_elementwise_maximum(fabsf(x[0]), fabsf(x[1])), most);
    most = __builtin_elementwise_maximum(__builtin_elementwise_maximum(fabsf(x[2]), fabsf(x[3])), most);
    least = fminf(fminf(fabsf(x[0]), fabsf(x[1])), least);
    least = fminf(fminf(fabsf(x[2]), fabsf(x[3])), least);
  }
};
__device__ __forceinline__ bool any_below(const f32x4& x, float least) {
  bool below = false;
#pragma unroll
  for (int e = 0; e < 4; ++e) below |= x[e] != 0.f && fabsf(x[e]) < least;
  return below;
}
// Of a row of Q or K: its logits are not those of the parts where the other operand's row has large numbers, or at all.
constexpr int kSmallNumbers = 1, kLargeNumbers = 2;
// ... of the pieces first, first + step, ... of `raw`
template <int N>
__device__ __forceinline__ int odd_numbers(const f32x4 (&raw)[N], int first, int step) {
  Extremes seen;
  int odd = 0;
#pragma unroll
  for (int p = 0; p < step; ++p)
    if (p == first) {
#pragma unroll
      for (int c = p; c < N; c += step) seen.see(raw[c]);
      if (seen.least < kSmallestSplit) {
#pragma unroll
        for (int c = p; c < N; c += step) odd |= any_below(raw[c], kSmallestSplit) ? kSmallNumbers : 0;
      }
    }
  return seen.most > kLargestRow ? odd | kLargeNumbers : odd;
}

// The 16 logits of a lane in plain arithmetic.  own(c): the piece c of four elements of the lane's own row; other(row, c): of the row
// (of the tile's 32) that register i belongs to.
template <int D, typename OwnFn, typename OtherFn>
__device__ __forceinline__ f32x16 plain_logits(int h, OwnFn own, OtherFn other) {
  f32x16 s;
#pragma unroll
  for (int i = 0; i < 16; ++i) s[i] = 0.f;
#pragma unroll 1
  for (int c = 0; c < D / 4; ++c) {
    const f32x4 x = own(c);
    asm volatile("" : "+v"(h));  // (no addresses kept from round to round: the registers are those of the products)
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const f32x4 y = other(8 * (i >> 2) + 4 * h + (i & 3), c);
#pragma unroll
      for (int e = 0; e < 4; ++e) s[i] = fmaf(x[e], y[e], s[i]);
      if (i % 4 == 3) __builtin_amdgcn_sched_barrier(0);  // (no more registers than the rest of the kernel has)
    }
  }
  return s;
}

// NW waves per workgroup, which has 32 RB query rows: wave w takes the rows 32 (w % RB) .. and every P-th key tile from
// w / RB on.  The RB waves of a part share its K and its V tile, in buffers of their own: V(t) is under way while the
// logits of tile t and their exponentials are formed, K(t + P) during the products with V(t).  A tile takes a wave 96 matrix ops
// (d = 128) of 32 cycles and about a thousand vector instructions, most of them for cutting K and V.  A wave alone on its SIMD
// issues a vector instruction every six cycles, two of them one every three, so registers are held to what two waves can have.
// 32 heads x 1000 rows x 128: 80 us (8.2 GFLOP = 102 TFLOP/s of fp32 products, of which a large fp32 matrix product reaches
// 154; on the fp32 instruction 103 us); 849 x 210: 152 (217).
template <int D, bool WITH_O, int RB, int NW>
__global__ __launch_bounds__(NW * 64, D == 64 && RB == 2 ? 3 : (RB == 1 && NW == 4 ? 1 : 2)) void attn_f32_kernel(
    const float* __restrict__ Q, const float* __restrict__ K, const float* __restrict__ V,
    AttnRect rc, int GQ, int nqb, float* __restrict__ O, float* __restrict__ LSE2, float scale_log2e) {
  constexpr int C16 = D / 16, DB = D / 32, kTileBytes = kRows * D * 4, P = NW / RB, BM = kRows * RB, NT = NW * 64;
  __shared__ __attribute__((aligned(1024))) char smem[2 * P * kTileBytes];
  __shared__ float m_s[NW][kRows], l_s[NW][kRows];
  __shared__ bool again;
  __shared__ int odd_rows[BM];
  const auto arrived = [] {  // this wave's loads, and those of the waves it shares tiles with
    if (RB == 1) { wait_vm<0>(); wait_lds(); }
    else wait_vm_barrier<0>();
  };

  int g, rank;
  if (!ordered_item(GQ, nqb, g, rank)) return;
  const int qb = rc.first_row / BM + nqb - 1 - rank;
  const int n = rc.m, row0 = qb * BM;
  const int gk = g / rc.kv_group;  // the K/V head this query head reads
  const int off = rc.off_heads ? rc.off_heads[gk] : 0;
  if (off < 0) {  // a head the caller's precondition excludes: its rows are flagged
    if (WITH_O)
      for (int e = threadIdx.x; e < min(BM, n - row0) * D; e += NT)
        O[((size_t)g * n + row0) * D + e] = __int_as_float(0x7FC00000);
    return;
  }
  const int nk = off + n;
  const float* Kg = K + (size_t)gk * rc.kv_stride * D;
  const float* Vg = V + (size_t)gk * rc.kv_stride * D;
  const int ntiles = (off + min(n, row0 + BM) - 1) / kRows + 1;

  // The whole block.  `careful`: the logits and products of operands without parts in plain arithmetic, tile by tile (a block
  // takes about twice the time, a tile that has them four times; a number without parts in V costs its key 500 instructions).
  const auto pass = [&](auto careful_) __attribute__((always_inline)) {
    constexpr bool careful = decltype(careful_)::value;
    int tid = threadIdx.x;
    if (careful) asm volatile("" : "+v"(tid));  // (nothing lives on from one pass to the other)
    const int lane = tid & 63, l32 = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), block = wave % RB, part = wave / RB;
    const int wrow0 = row0 + kRows * block;
    lds_char* const kbuf = (lds_char*)smem + part * 2 * kTileBytes;
    lds_char* const vbuf = kbuf + kTileBytes;  // (without outputs: a second K buffer)
    const int nt_wave = wrow0 < n ? (off + min(n, wrow0 + kRows) - 1) / kRows + 1 : 0;  // tiles this wave's rows see
    // chunk 4c + 2h + e of row l32: the swizzle reaches the low four chunk bits, so c and e are an exclusive or with the first one's place
    const uint32_t koff = l32 * D * 4 + (((2 * h) ^ tile_swizzle<false>(l32)) << 4);
    const int voff[2] = {4 * h * D * 4 + l32 * 4 + h * 128, 4 * h * D * 4 + l32 * 4 + (1 - h) * 128};
    const int newest = off + wrow0 + l32;  // newest key this lane's row sees
    const float* const q_row = Q + ((size_t)g * n + min(wrow0 + l32, n - 1)) * D;
    if (part < ntiles) fetch_tile<D, false>(Kg, part * kRows, nk, kbuf, block, RB);
    // Q (B operand): lane (query l32, half h) holds the elements 16c + 8h .. + 7; a careful pass splits them for every tile again, which
    // leaves it registers for the plain arithmetic (memory for spilled ones is paid for by every workgroup, at its start)
    Parts qf[careful ? 1 : C16];
    int odd = 0;  // kSmallNumbers ... of this part's share of the row
    const auto query = [&](int c) -> Parts {
      if constexpr (!careful) return qf[c];
      const float* qr = q_row + 16 * c + 8 * h;
      asm volatile("" : "+v"(qr));
      return split(*reinterpret_cast<const f32x4*>(qr), *reinterpret_cast<const f32x4*>(qr + 4));
    };
    if constexpr (careful) {
      odd = odd_rows[kRows * block + l32];
    } else {
      const float* qr = q_row + 8 * h;
      f32x4 raw[2 * C16];
#pragma unroll
      for (int c = 0; c < 2 * C16; ++c) raw[c] = *reinterpret_cast<const f32x4*>(qr + 16 * (c >> 1) + 4 * (c & 1));
#pragma unroll
      for (int c = 0; c < C16; ++c) qf[c] = split(raw[2 * c], raw[2 * c + 1]);
#pragma unroll
      for (int c = 0; c < C16; ++c) asm volatile("" : "+v"(qf[c].high.x));  // formed here, not in every round of the loop
      odd = odd_numbers(raw, part, P);
      if (tid < BM) odd_rows[tid] = 0;
      if (tid == 0) again = false;
    }

    f32x16 oacc[WITH_O ? DB : 1];
#pragma unroll
    for (int db = 0; db < (WITH_O ? DB : 1); ++db)
#pragma unroll
      for (int i = 0; i < 16; ++i) oacc[db][i] = 0.f;
    float m = kLowest, l = 0.f;

    for (int t = part, step = 0; t < ntiles + part; t += P, ++step) {  // (the parts take the same number of steps)
      const int key0 = t * kRows;
      const bool mine = t < nt_wave;
      lds_char* const kt = WITH_O || step % 2 == 0 ? kbuf : vbuf;
      arrived();  // K tile t; the other buffer is free
      if (WITH_O && t < ntiles) fetch_tile<D, true>(Vg, key0, nk, vbuf, block, RB);
      if (!WITH_O && t + P < ntiles) fetch_tile<D, false>(Kg, key0 + P * kRows, nk, kt == kbuf ? vbuf : kbuf, block, RB);
      Parts pf[2];
      if (mine) {
        f32x16 s, rest;
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] = rest[i] = 0.f;
        const auto read = [&](int c, f32x4& a, f32x4& b) {
          const uint32_t at = (uint32_t)(size_t)kt + koff;
          a = lds_read4((const lds_char*)(size_t)(at ^ (c & 3) << 6) + (c >> 2) * 256);
          b = lds_read4((const lds_char*)(size_t)(at ^ ((c & 3) << 6 | 16)) + (c >> 2) * 256);
        };
        f32x4 a, b;
        Extremes keys;
        read(0, a, b);
#pragma unroll
        for (int c = 0; c < C16; ++c) {
          const Parts kp = split(a, b);
          if constexpr (careful) { keys.see(a); keys.see(b); }
          if (c + 1 < C16) read(c + 1, a, b);
          multiply(kp, query(c), s, rest);
          __builtin_amdgcn_sched_barrier(0);  // (more pieces at once do not fit the registers)
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] += rest[i];
        if constexpr (careful) {
          const bool plain_row = (odd & kLargeNumbers) || ((odd & kSmallNumbers) && __any(keys.most > kLargestRow));
          bool some = plain_row;
#pragma unroll
          for (int i = 0; i < 16; ++i) some |= !finite(s[i]);
          if (__any(some)) {
            const f32x16 exact = plain_logits<D>(
                h, [&](int c) { return *reinterpret_cast<const f32x4*>(q_row + 4 * c); },
                [&](int row, int c) { return lds_read4(kt + row * D * 4 + ((c ^ tile_swizzle<false>(row)) << 4)); });
#pragma unroll
            for (int i = 0; i < 16; ++i) s[i] = plain_row || !finite(s[i]) ? exact[i] : s[i];
          }
        }
        if (key0 + kRows - 1 > off + wrow0) {  // the tile reaches past the block's first row
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
        for (int i = 0; i < 16; ++i) s[i] = __builtin_amdgcn_exp2f((s[i] - m) * scale_log2e);
        float sum[4];  // (of few terms each before they join the row's)
#pragma unroll
        for (int i = 0; i < 4; ++i) sum[i] = (s[4 * i] + s[4 * i + 1]) + (s[4 * i + 2] + s[4 * i + 3]);
        l += (sum[0] + sum[1]) + (sum[2] + sum[3]);
        if (WITH_O) {
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            float x[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) x[i] = s[8 * j + i];
            pf[j] = split(x);
          }
        }
      }
      if constexpr (WITH_O) {
        arrived();  // V tile t; every wave that shares K tile t has read it
        if (t + P < ntiles) fetch_tile<D, false>(Kg, key0 + P * kRows, nk, kbuf, block, RB);
        if (mine) {
          constexpr int NV = 2 * DB;  // (columns 32 db .., step j), j fastest
          float x[8];
          const auto read = [&](int v) {
            const int db = v >> 1, j = v & 1;
#pragma unroll
            for (int i = 0; i < 8; ++i)
              x[i] = lds_read1(vbuf + voff[db & 1] + (db >> 1) * 256 + (16 * j + 8 * (i >> 2) + (i & 3)) * D * 4);
          };
          float up = 1.f, down = 1.f;  // careful: small numbers are split as multiples where that makes none too large
          if constexpr (careful) {
            float most = 0.f;
#pragma unroll 1
            for (int u = 0; u < D / 8; ++u) {
              const f32x4 y = lds_read4(vbuf + u * 1024 + lane * 16);
#pragma unroll
              for (int e = 0; e < 4; ++e) most = fmaxf(most, finite(y[e]) ? fabsf(y[e]) : 0.f);
            }
            if (wave_max(most) <= 0x1p60f) { up = 0x1p64f; down = 0x1p-64f; }
          }
          f32x16 o;  // of this tile alone: rounded at its own size before it joins the others
          read(0);
#pragma unroll
          for (int v = 0; v < NV; ++v) {
            if (v % 2 == 0) {
#pragma unroll
              for (int i = 0; i < 16; ++i) o[i] = 0.f;
            }
            if constexpr (careful) {
#pragma unroll
              for (int i = 0; i < 8; ++i) x[i] = has_parts(x[i] * up) ? x[i] * up : 0.f;
            }
            const Parts vp = split(x);
            if (v + 1 < NV) read(v + 1);
            multiply(vp, pf[v & 1], o, o);
            if (v % 2 == 1) {
#pragma unroll
              for (int i = 0; i < 16; ++i) oacc[v >> 1][i] += careful ? o[i] * down : o[i];
            }
            __builtin_amdgcn_sched_barrier(0);
          }
          if constexpr (careful) {
            // what was left out: p v for every v without parts, by the rows that see its key
#pragma unroll 1
            for (int key = 0; key < kRows; ++key) {
              const lds_char* const v_row = vbuf + key * D * 4;
              bool some = !has_parts(lds_read1(v_row + lane * 4) * up);
              if (D == 128) some |= !has_parts(lds_read1(v_row + 256 + lane * 4) * up);
              if (!__any(some)) continue;
              const int at = 4 * (key >> 3) + (key & 3);  // its register, in the lanes of half (key >> 2) & 1
              float p = 0.f;
#pragma unroll
              for (int j = 0; j < 2; ++j)  // (put together again for every key: no registers for sixteen numbers)
                asm volatile("" : "+v"(pf[j].high.x), "+v"(pf[j].high.y), "+v"(pf[j].high.z), "+v"(pf[j].high.w), "+v"(pf[j].middle.x),
                             "+v"(pf[j].middle.y), "+v"(pf[j].middle.z), "+v"(pf[j].middle.w), "+v"(pf[j].low.x),
                             "+v"(pf[j].low.y), "+v"(pf[j].low.z), "+v"(pf[j].low.w));
#pragma unroll
              for (int i = 0; i < 16; ++i) p = at == i ? joined(pf[i >> 3], i & 7) : p;
              const float theirs = __shfl_xor(p, 32);
              p = ((key >> 2) & 1) == h ? p : theirs;
#pragma unroll
              for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int i4 = 0; i4 < 4; ++i4) {
                  const f32x4 v4 = lds_read4(v_row + (((8 * db + 2 * i4 + h) ^ tile_swizzle<true>(key)) << 4));
#pragma unroll
                  for (int e = 0; e < 4; ++e)
                    if (key0 + key <= newest && !has_parts(v4[e] * up)) oacc[db][4 * i4 + e] = fmaf(p, v4[e], oacc[db][4 * i4 + e]);
                  __builtin_amdgcn_sched_barrier(0);
                }
            }
          }
        }
      }
    }
    wait_vm_barrier<0>();  // the buffers are reused below
    if (!careful && odd) { atomicOr(&odd_rows[kRows * block + l32], odd); again = true; }

    // ---- the parts' sums
    l = across_rows(l, OpAdd(), false, true);
    if (h == 0) { m_s[wave][l32] = m; l_s[wave][l32] = l; }
    __syncthreads();
    float mall = m_s[block][l32];
#pragma unroll
    for (int w = 1; w < P; ++w) mall = fmaxf(mall, m_s[block + RB * w][l32]);
    float lall = 0.f;
#pragma unroll
    for (int w = 0; w < P; ++w) lall += l_s[block + RB * w][l32] * exp2f((m_s[block + RB * w][l32] - mall) * scale_log2e);
    if (part == 0 && h == 0 && wrow0 + l32 < n) {
      float* const lse = LSE2 + (size_t)g * n + wrow0 + l32;
      // (a sum that was finite stands, whatever the outputs are: the scores' logits are those it was formed from)
      if (!careful || odd || !finite(*lse)) *lse = fmaf(mall, scale_log2e, log2f(lall));
      if (!careful && !(lall > 0.f && lall < INFINITY)) again = true;
    }
    if constexpr (WITH_O) {
      const float f = exp2f((m - mall) * scale_log2e) / lall;
      // a tile's room per wave now takes its outputs, [query][d], chunks swizzled as in a tile
      lds_char* const strip = (lds_char*)smem + wave * kTileBytes;
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
      for (int u = tid; u < BM * CPR; u += NT) {
        const int r = u / CPR, c = u % CPR;
        if (row0 + r >= n) break;
        const lds_char* p = (const lds_char*)smem + r * D * 4 + ((c ^ tile_swizzle<false>(r)) << 4);
        f32x4 a = lds_read4(p);
        if constexpr (P > 1) a += lds_read4(p + RB * kTileBytes);
#pragma unroll
        for (int w = 2; w < P; w += 2) a += lds_read4(p + RB * w * kTileBytes) + lds_read4(p + RB * (w + 1) * kTileBytes);
        *reinterpret_cast<f32x4*>(O + ((size_t)g * n + row0 + r) * D + c * 4) = a;
        if constexpr (!careful) {
          Extremes seen;
          seen.see(a);
          if (!(seen.most <= kLargest) || (seen.least < kSmallestSum && any_below(a, kSmallestSum))) again = true;
        }
      }
    }
  };
  pass(std::false_type{});
  __syncthreads();
  if (again) pass(std::true_type{});
}

// One workgroup per 32 keys, whose K rows stay in registers; wave w takes every NW-th tile of 32
// query rows of the head's kv_group query heads.  `accumulate`: the result is added to `decay`
// times what scores[] holds (a chunk: the cached tokens' older scores, decayed by alpha^m);
// otherwise it replaces it.
template <int D, int NW>
__global__ __launch_bounds__(NW * 64, D == 64 ? 3 : 2) void scores_f32_kernel(
    const float* __restrict__ Q, const float* __restrict__ K, const float* __restrict__ LSE2,
    AttnRect rc, int G, int ncb, int first_row, float log2_alpha, const float* __restrict__ alpha_heads,
    float* __restrict__ scores, int s_stride, bool accumulate, float decay, float scale_log2e) {
  constexpr int C16 = D / 16, kTileBytes = kRows * D * 4;
  __shared__ __attribute__((aligned(1024))) char smem[NW * kTileBytes];
  __shared__ float part[NW][kRows];
  __shared__ bool again;
  __shared__ int odd_keys[kRows];
  int g, rank;
  if (!ordered_item(G, ncb, g, rank)) return;
  const int c0 = rank * kRows;  // the oldest keys have the most rows
  const int n = rc.m;
  const int off = rc.off_heads ? rc.off_heads[g] : 0;
  const int nk = off + n;
  if (off < 0 || c0 >= nk) return;
  head_window(alpha_heads, g, n, first_row, log2_alpha);
  const float* Qg = Q + (size_t)g * rc.kv_group * n * D;  // the group's rows lie one head after the other
  const float* lg = LSE2 + (size_t)g * rc.kv_group * n;
  const float* const Kg = K + (size_t)g * rc.kv_stride * D;
  const int t0 = max(max(c0 - off, first_row), 0) / kRows;  // first row tile that counts
  const int nt = (n + kRows - 1) / kRows - t0;              // tiles per query head
  const int work = nt * rc.kv_group;

  // The sum of key c0 + tid, for tid < 32.  `careful`: logits of operands without parts in plain arithmetic.
  const auto total = [&](auto careful_) __attribute__((always_inline)) -> float {
    constexpr bool careful = decltype(careful_)::value;
    int tid = threadIdx.x;
    if (careful) asm volatile("" : "+v"(tid));  // (nothing lives on from one pass to the other)
    const int lane = tid & 63, l32 = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    lds_char* const qt = (lds_char*)smem + wave * kTileBytes;
    auto fetch = [&](int f) {
      const int hq = f / nt, t = t0 + f % nt;
      fetch_tile<D, false>(Qg + (size_t)hq * n * D, t * kRows, n, qt);
    };
    if (wave < work) fetch(wave);
    Parts kf[careful ? 1 : C16];  // A operand: lane (key l32, half h) holds the elements 16c + 8h .. + 7
    int odd = 0;  // kSmallNumbers ... of this wave's share of the lane's key
    uint32_t small_keys = 0, large_keys = 0;
    const float* const k_row = Kg + (size_t)min(c0 + l32, nk - 1) * D + 8 * h;
    const auto key_parts = [&](int c) -> Parts {
      if constexpr (!careful) return kf[c];
      const float* kr = k_row + 16 * c;
      asm volatile("" : "+v"(kr));
      return split(*reinterpret_cast<const f32x4*>(kr), *reinterpret_cast<const f32x4*>(kr + 4));
    };
    if constexpr (careful) {
      small_keys = (uint32_t)__ballot(odd_keys[l32] & kSmallNumbers);
      large_keys = (uint32_t)__ballot(odd_keys[l32] & kLargeNumbers);
    } else {
      f32x4 raw[2 * C16];
#pragma unroll
      for (int c = 0; c < 2 * C16; ++c) raw[c] = *reinterpret_cast<const f32x4*>(k_row + 16 * (c >> 1) + 4 * (c & 1));
#pragma unroll
      for (int c = 0; c < 2 * C16; ++c) asm volatile("" : "+v"(raw[c]));  // waited for here, not in every round of the loop
#pragma unroll
      for (int c = 0; c < C16; ++c) kf[c] = split(raw[2 * c], raw[2 * c + 1]);
      odd = odd_numbers(raw, wave, NW);
      if (tid == 0) again = false;
      if (tid < kRows) odd_keys[tid] = 0;
    }
    int qoff[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) qoff[i] = l32 * D * 4 + (((4 * (i >> 1) + 2 * h + (i & 1)) ^ tile_swizzle<false>(l32)) << 4);
    float acc[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.f;

    for (int f = wave; f < work; f += NW) {
      const int hq = f / nt, r = (t0 + f % nt) * kRows + l32;
      float lse = lg[(size_t)hq * n + min(r, n - 1)];
      asm volatile("" : "+v"(lse));  // with the tile: everything has arrived
      wait_vm<0>();
      f32x16 s, rest;
#pragma unroll
      for (int i = 0; i < 16; ++i) s[i] = rest[i] = 0.f;
      Extremes queries;
#pragma unroll
      for (int c = 0; c < C16; ++c) {
        const lds_char* p = qt + (c >> 2) * 256;
        const f32x4 a = lds_read4(p + qoff[2 * (c & 3)]), b = lds_read4(p + qoff[2 * (c & 3) + 1]);
        if constexpr (careful) { queries.see(a); queries.see(b); }
        multiply(key_parts(c), split(a, b), s, rest);
      }
#pragma unroll
      for (int i = 0; i < 16; ++i) s[i] += rest[i];
      if constexpr (careful) {
        const auto key_of = [&](int i) { return 8 * (i >> 2) + 4 * h + (i & 3); };
        const uint32_t plain_keys = large_keys | (__any(queries.most > kLargestRow) ? small_keys : 0);
        const auto plain = [&](int i) { return (plain_keys >> key_of(i) & 1) || !finite(s[i]); };
        bool some = false;
#pragma unroll
        for (int i = 0; i < 16; ++i) some |= plain(i);
        if (__any(some && lse == lse)) {  // (a row whose sum is NaN stays so)
          const f32x16 exact = plain_logits<D>(
              h, [&](int c) { return lds_read4(qt + l32 * D * 4 + ((c ^ tile_swizzle<false>(l32)) << 4)); },
              [&](int row, int c) { return *reinterpret_cast<const f32x4*>(Kg + (size_t)min(c0 + row, nk - 1) * D + 4 * c); });
#pragma unroll
          for (int i = 0; i < 16; ++i) s[i] = plain(i) ? exact[i] : s[i];
        }
      }
      wait_lds();
      if (f + NW < work) fetch(f + NW);
      // exponent offset of row r: lse_r - (n-1-r) log2(alpha); rows past the end, and rows whose
      // weight is exactly 0 in fp32 (before first_row), add nothing
      const bool counts = r < n && r >= first_row;
      const float w = (float)(n - 1 - r) * log2_alpha;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const float p = exp2f(fmaf(s[i], scale_log2e, -lse) + w);
        acc[i] += counts && c0 + 8 * (i >> 2) + 4 * h + (i & 3) <= off + r ? p : 0.f;
      }
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      acc[i] = group_sum<32>(acc[i]);  // over the 32 rows held by the lanes of one half
      if (l32 == 0) part[wave][8 * (i >> 2) + 4 * h + (i & 3)] = acc[i];
    }
    __syncthreads();
    if (!careful && odd) { atomicOr(&odd_keys[l32], odd); again = true; }
    float sum = 0.f;
    if (tid < kRows) {
#pragma unroll
      for (int w = 0; w + 3 < NW; w += 4) sum += (part[w][tid] + part[w + 1][tid]) + (part[w + 2][tid] + part[w + 3][tid]);
      if constexpr (NW < 4) sum = NW == 1 ? part[0][tid] : part[0][tid] + part[NW - 1][tid];
    }
    return sum;
  };
  const int tid = threadIdx.x;
  const bool live = tid < kRows && c0 + tid < nk;
  float* const out = scores + (size_t)g * s_stride + c0 + tid;
  float sum = total(std::false_type{});
  const float older = live && accumulate ? *out : 0.f;
  if (live) {
    *out = accumulate ? fmaf(decay, older, sum) : sum;
    if (!(sum < INFINITY)) again = true;
  }
  __syncthreads();
  if (!again) return;
  sum = total(std::true_type{});
  if (live) *out = accumulate ? fmaf(decay, older, sum) : sum;
}

// ---- short prompts -------------------------------------------------------------------------
// A tile of 32 rows is a chain of 96 matrix ops (d = 128) of 32 cycles and the vector work between them, 3000 cycles and more, whatever
// the prompt has of it.  A short prompt of few heads is done sooner by plain arithmetic: a workgroup per attention row, then one
// per key (square geometry only).
constexpr int kShortRows = 384;  // of a prompt, at most

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
// about constant, but for one head, whose rows grow longer than that takes, and for many heads of a few rows of d = 128 (us per call, rows / tiles:
// d = 128, 1 head x 239 rows 25.7 / 28.9, x 299 31.5 / 33.1, x 359 38.3 / 34.6, 2 x 188 26.2 / 28.9, x 226 30.9 / 29.9, 4 x 140 24.8 / 28.6, x 178
// 29.3 / 29.8, 8 x 89 20.6 / 23.2, x 112 24.8 / 22.9, 32 x 35 17.9 / 20.6, 60 x 23 17.8 / 20.9, 120 x 14 17.6 / 18.8, 300 x 6 17.4 / 19.0, x 7 19.3 /
// 19.3, 1000 x 2 17.6 / 19.9, x 3 22.4 / 20.4; d = 64, 1 x 268 19.5 / 22.5, x 358 22.1 / 22.4, x 448 26.2 / 24.9, 2 x 225 19.1 / 21.4, x 282 22.4 / 22.6,
// 4 x 213 22.5 / 22.4, 16 x 74 14.6 / 17.9, 32 x 44 12.8 / 15.8, 120 x 18 12.0 / 14.8, 300 x 10 12.6 / 15.0, 1000 x 4 13.9 / 15.5).
static bool short_prompt(int G, const AttnRect& rc, int d) {
  const double rows = (double)G * rc.kv_group * rc.m, work = rows * rows * rc.m;
  if (rc.off_heads) return false;
  return d == 64 ? rc.m <= kShortRows && work <= 90e6 : rc.m <= 320 && rows <= 2100 && work <= 45e6;
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
  const auto blocks = [&](int rows) { return (rc.m + rows - 1) / rows - rc.first_row / rows; };  // row blocks to compute
#define A2SF_ATTN_F32(D, WO, RB, NW)                                                                  \
  hipLaunchKernelGGL((attn_f32_kernel<D, WO, RB, NW>), dim3(ordered_grid(GQ, blocks(kRows * RB))), dim3(NW * 64), 0, st, \
                     q, k, v, rc, GQ, blocks(kRows * RB), o, lse2, scale_log2e)
#define A2SF_ATTN_F32_64(WO)                             \
  do {                                                   \
    if (tiles == 1) A2SF_ATTN_F32(64, WO, 1, 1);         \
    else if (all <= 320 && tiles >= 8) A2SF_ATTN_F32(64, WO, 1, 8); \
    else if (all <= 1024 && tiles == 2) A2SF_ATTN_F32(64, WO, 1, 2); \
    else if (all <= 1024) A2SF_ATTN_F32(64, WO, 1, 4);   \
    else A2SF_ATTN_F32(64, WO, 2, 4);                    \
  } while (0)
#define A2SF_ATTN_F32_128(WO)                            \
  do {                                                   \
    if (tiles == 1) A2SF_ATTN_F32(128, WO, 1, 1);        \
    else if (all <= one_block && tiles == 2) A2SF_ATTN_F32(128, WO, 1, 2); \
    else if (all <= one_block) A2SF_ATTN_F32(128, WO, 1, 4); \
    else A2SF_ATTN_F32(128, WO, 2, 4);                   \
  } while (0)
  // Two blocks of rows per workgroup share a tile's loads and put two waves onto every SIMD; while the blocks are few, the chain
  // of a row's tiles counts, and one block takes all waves (us, one block with eight waves / with four / two blocks: d = 64,
  // 76 blocks of 32 rows 12.7 / 14.0 / 22.4, 228 14.1 / 17.2 / 27.2, 580 33.5 / 28.0 / 39.8, 1000 35.4 / 25.8 / 28.8, 2000 86.6 /
  // 66.3 / 61.2, 2820 178 / 147 / 133, but 80 of two tiles 8.5 / 7.7; d = 128, four waves / two blocks: 38 blocks 41.4 / 73.0, 377 43.6 / 59.7, 752 105.7 / 105.2,
  // 760 81.4 / 66.7, 1024 102 / 80, 5943 270 / 152.  Eight waves of d = 128 have no registers for the parts).
  const long long all = (long long)GQ * blocks(kRows);
  const int tiles = ((rc.off_heads ? rc.kv_stride : rc.m) + kRows - 1) / kRows;  // of the newest row, at most
  // One tile in all: one wave per workgroup, which leaves room for many (us per call, four waves / one: d = 64, 400 heads x 15 rows 17.3 / 15.7, 800 x
  // 15 28.0 / 17.1, 2000 x 32 49.4 / 32.8; d = 128, 400 x 15 29.9 / 21.3, 800 x 32 50.0 / 33.9, 2000 x 6 68.1 / 33.3; scores included).  Two: two waves
  // (four / two: d = 64, 400 x 64 27.4 / 21.5; d = 128, 200 x 64 31.7 / 23.7, 60 x 64 21.8 / 20.7), but two blocks of rows where those are
  // taken (two blocks / two waves: d = 64, 2000 x 64 48.6 / 52.0; d = 128, 400 x 64 31.5 / 37.0).
  // d = 128, 513 to 640 blocks: one block per workgroup takes a third round, which only long chains are worth (us per call, one block / two: 64 x 320
  // 65.6 / 56.2, 180 x 96 50.8 / 40.6, 32 x 610 74.2 / 70.5, but 20 x 870 78.7 / 83.1, 9 x 1900 111 / 141).
  const long long one_block = tiles > 24 ? 640 : 512;
  if (d == 64) {
    if (o) A2SF_ATTN_F32_64(true); else A2SF_ATTN_F32_64(false);
  } else {
    if (o) A2SF_ATTN_F32_128(true); else A2SF_ATTN_F32_128(false);
  }
#undef A2SF_ATTN_F32_64
#undef A2SF_ATTN_F32_128
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
#define A2SF_SCORES_F32(D, NW)                                                                        \
  hipLaunchKernelGGL((scores_f32_kernel<D, NW>), dim3(ordered_grid(G, ncb)), dim3(NW * 64), 0, st, q, k, lse2, rc, G, ncb, first, \
                     l2a, alpha_heads, scores, s_stride, accumulate, decay, scale_log2e)
  // Eight waves where the keys are few and every wave has a tile (us, eight waves / four: d = 128, 38 blocks of 32 keys x 33 tiles 20.7
  // / 27.8, 94 x 376 150 / 230, 256 x 32 22.6 / 27.1, but 264 x 2 17.3 / 11.1, 377 x 3 17.8 / 11.5, 1024 x 3 36 / 22; d = 64, 228 x
  // 8 7.8 / 8.6, 111 x 24 11.5 / 17.5, 580 x 29 25.9 / 21.0).
  // One tile of rows: one wave (us per call, four / one, chunks of 2 rows behind 150, d = 128: 300 heads 74 / 56, 1307 heads 211 / 138; 32 heads 33.7 /
  // 32.7).  Two: two waves (four / two, chunks of 60 rows behind 200: 300 heads 124 / 107, 1307 heads 412 / 318; 32 heads 46.5 / 45.5).
  const int tiles = ((rc.m + kRows - 1) / kRows - first / kRows) * rc.kv_group;
  const bool few = (long long)G * ncb <= 320 && tiles >= 8;
  if (d == 64) {
    if (tiles == 1) A2SF_SCORES_F32(64, 1); else if (tiles == 2) A2SF_SCORES_F32(64, 2); else if (few) A2SF_SCORES_F32(64, 8); else A2SF_SCORES_F32(64, 4);
  } else {
    if (tiles == 1) A2SF_SCORES_F32(128, 1); else if (tiles == 2) A2SF_SCORES_F32(128, 2); else if (few) A2SF_SCORES_F32(128, 8); else A2SF_SCORES_F32(128, 4);
  }
#undef A2SF_SCORES_F32
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
