// Device-side helpers shared by the A2SF kernels (gfx950, wave64).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace a2sf {

typedef uint16_t bf16_t;  // storage type of bf16 elements (bit pattern)

constexpr int kWave = 64;
constexpr int kThreads = 256;  // threads per workgroup, where a kernel does not name its own number
constexpr int kWaves = kThreads / kWave;

// ---- element conversion ----------------------------------------------------------------
__device__ __forceinline__ float bf16_to_f32(uint32_t bits16) { return __uint_as_float(bits16 << 16); }

// round to nearest even; inputs are finite in every caller
__device__ __forceinline__ uint32_t f32_to_bf16(float x) {
  uint32_t u = __float_as_uint(x);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return u >> 16;
}

// two floats -> packed bf16 pair (lo in bits 0..15), hardware round-to-nearest-even
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  f32x2_t v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}

template <typename T> struct Elem;
template <> struct Elem<float> {
  static constexpr int kPerLane = 4;  // elements in one 16-byte access
  __device__ static __forceinline__ void unpack(const uint4& r, float* f) {
    f[0] = __uint_as_float(r.x); f[1] = __uint_as_float(r.y);
    f[2] = __uint_as_float(r.z); f[3] = __uint_as_float(r.w);
  }
  __device__ static __forceinline__ void store(float* p, float x) { *p = x; }
};
template <> struct Elem<bf16_t> {
  static constexpr int kPerLane = 8;
  __device__ static __forceinline__ void unpack(const uint4& r, float* f) {
    f[0] = __uint_as_float(r.x << 16); f[1] = __uint_as_float(r.x & 0xFFFF0000u);
    f[2] = __uint_as_float(r.y << 16); f[3] = __uint_as_float(r.y & 0xFFFF0000u);
    f[4] = __uint_as_float(r.z << 16); f[5] = __uint_as_float(r.z & 0xFFFF0000u);
    f[6] = __uint_as_float(r.w << 16); f[7] = __uint_as_float(r.w & 0xFFFF0000u);
  }
  __device__ static __forceinline__ void store(bf16_t* p, float x) { *p = (bf16_t)f32_to_bf16(x); }
};

// 16 bytes of packed elements from EPL floats (inverse of Elem<T>::unpack)
__device__ __forceinline__ uint4 pack16(const float* f, float) {
  return make_uint4(__float_as_uint(f[0]), __float_as_uint(f[1]), __float_as_uint(f[2]), __float_as_uint(f[3]));
}
__device__ __forceinline__ uint4 pack16(const float* f, bf16_t) {
  return make_uint4(pack_bf16(f[0], f[1]), pack_bf16(f[2], f[3]), pack_bf16(f[4], f[5]), pack_bf16(f[6], f[7]));
}

// ---- lane exchanges ---------------------------------------------------------------------
// Reductions over the wave stay in the vector pipe: inside a row of 16 lanes DPP lane
// permutations folded into the operation (quad swaps, then mirrors inside half rows and rows:
// a mirror pairs each lane with one holding the other half's partial result), across rows the
// two swap instructions of gfx950 (odd with even rows of 16 lanes, upper with lower half of
// the wave).  A butterfly through the LDS crossbar (ds_bpermute) costs ~100 cycles of latency
// per step instead of a handful.
template <int CTRL>
__device__ __forceinline__ float dpp_move(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_move_u32(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, false);
}
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
// the value of lane l ^ 16 / l ^ 32
__device__ __forceinline__ uint32_t lane_xor16_u32(uint32_t v) {
  const u32x2_t r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  return ((threadIdx.x >> 4) & 1) ? r[0] : r[1];   // r[0] = rows (0,0,2,2), r[1] = rows (1,1,3,3)
}
__device__ __forceinline__ uint32_t lane_xor32_u32(uint32_t v) {
  const u32x2_t r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return ((threadIdx.x >> 5) & 1) ? r[0] : r[1];   // r[0] = halves (lo, lo), r[1] = (hi, hi)
}
// op(v of this lane, v of the partner lane) for commutative op, both steps across rows
template <typename Op>
__device__ __forceinline__ float across_rows(float v, Op op, bool rows16, bool halves) {
  if (rows16) {
    const u32x2_t r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = op(__uint_as_float(r[0]), __uint_as_float(r[1]));
  }
  if (halves) {
    const u32x2_t r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = op(__uint_as_float(r[0]), __uint_as_float(r[1]));
  }
  return v;
}
struct OpAdd { __device__ __forceinline__ float operator()(float a, float b) const { return a + b; } };
struct OpMax { __device__ __forceinline__ float operator()(float a, float b) const { return fmaxf(a, b); } };

// Sum over aligned groups of N consecutive lanes (N = 8, 16, 32 or 64); every lane of a
// group gets the group's total.
template <int N>
__device__ __forceinline__ float group_sum(float v) {
  v += dpp_move<0xB1>(v);                  // quad_perm [1,0,3,2]
  v += dpp_move<0x4E>(v);                  // quad_perm [2,3,0,1]
  if (N >= 8) v += dpp_move<0x141>(v);     // row_half_mirror
  if (N >= 16) v += dpp_move<0x140>(v);    // row_mirror
  return across_rows(v, OpAdd(), N >= 32, N >= 64);
}

// ---- ordering ---------------------------------------------------------------------------
// Monotone map float -> uint32 (larger float = larger key); -0 is folded onto +0.
__device__ __forceinline__ uint32_t ordered_key(float s) {
  uint32_t u = __float_as_uint(s + 0.0f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// The same without the keys 0 and all ones, which only a NaN of all bits set has: a selection marks slots with them.
__device__ __forceinline__ uint32_t score_key(float s) { return min(max(ordered_key(s), 1u), 0xFFFFFFFEu); }

// ---- wave / block reductions ------------------------------------------------------------
__device__ __forceinline__ float wave_max(float v) {
  v = fmaxf(v, dpp_move<0xB1>(v));
  v = fmaxf(v, dpp_move<0x4E>(v));
  v = fmaxf(v, dpp_move<0x141>(v));
  v = fmaxf(v, dpp_move<0x140>(v));
  return across_rows(v, OpMax(), true, true);
}
__device__ __forceinline__ float wave_sum(float v) { return group_sum<64>(v); }
__device__ __forceinline__ int wave_sum_i(int v) {
  uint32_t u = (uint32_t)v;
  u += dpp_move_u32<0xB1>(u);
  u += dpp_move_u32<0x4E>(u);
  u += dpp_move_u32<0x141>(u);
  u += dpp_move_u32<0x140>(u);
  u32x2_t r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  u = r[0] + r[1];
  r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return (int)(r[0] + r[1]);
}
__device__ __forceinline__ int wave_max_i(int v) {
  v = ::max(v, (int)dpp_move_u32<0xB1>((uint32_t)v));
  v = ::max(v, (int)dpp_move_u32<0x4E>((uint32_t)v));
  v = ::max(v, (int)dpp_move_u32<0x141>((uint32_t)v));
  v = ::max(v, (int)dpp_move_u32<0x140>((uint32_t)v));
  u32x2_t r = __builtin_amdgcn_permlane16_swap((uint32_t)v, (uint32_t)v, false, false);
  v = ::max((int)r[0], (int)r[1]);
  r = __builtin_amdgcn_permlane32_swap((uint32_t)v, (uint32_t)v, false, false);
  return ::max((int)r[0], (int)r[1]);
}
// lane `src` (the same for the whole wave) hands its value to every lane
__device__ __forceinline__ float wave_broadcast(float v, int src) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), __builtin_amdgcn_readfirstlane(src)));
}
__device__ __forceinline__ unsigned long long wave_min_u64(unsigned long long v) {
  uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
  const auto take = [&](uint32_t olo, uint32_t ohi) {
    const unsigned long long other = ((unsigned long long)ohi << 32) | olo;
    const unsigned long long mine = ((unsigned long long)hi << 32) | lo;
    if (other < mine) { lo = olo; hi = ohi; }
  };
  take(dpp_move_u32<0xB1>(lo), dpp_move_u32<0xB1>(hi));
  take(dpp_move_u32<0x4E>(lo), dpp_move_u32<0x4E>(hi));
  take(dpp_move_u32<0x141>(lo), dpp_move_u32<0x141>(hi));
  take(dpp_move_u32<0x140>(lo), dpp_move_u32<0x140>(hi));
  take(lane_xor16_u32(lo), lane_xor16_u32(hi));
  take(lane_xor32_u32(lo), lane_xor32_u32(hi));
  return ((unsigned long long)hi << 32) | lo;
}

// Block-wide reductions over 4 waves; `red` is a shared array of >= 8 floats / u64.
// All threads get the result.  Contain two barriers each.
__device__ __forceinline__ float block_max(float v, float* red) {
  v = wave_max(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
}
__device__ __forceinline__ float block_sum(float v, float* red) {
  v = wave_sum(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return (red[0] + red[1]) + (red[2] + red[3]);
}
__device__ __forceinline__ int block_sum_i(int v, int* red) {
  v = wave_sum_i(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return (red[0] + red[1]) + (red[2] + red[3]);
}
__device__ __forceinline__ unsigned long long block_min_u64(unsigned long long v,
                                                            unsigned long long* red) {
  v = wave_min_u64(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  unsigned long long a = red[0] < red[1] ? red[0] : red[1];
  unsigned long long b = red[2] < red[3] ? red[2] : red[3];
  return a < b ? a : b;
}

// ---- selection by threshold counts --------------------------------------------------------
// What the waves of a search share (one wave alone needs nothing).
template <int NW>
struct SelectSmem {
  int cnt[2][NW * 8];  // per wave: counts of up to eight thresholds; two sets, so a round needs one barrier
  int lo[NW], hi[NW];
};
template <>
struct SelectSmem<1> {};

// Sum over the waves of the counts that every wave has put into cnt[wave * 8 + i], i < 8: the
// lanes i = lane % 8 get the total of threshold i.
template <int NW>
__device__ __forceinline__ int sum_counts(const int* cnt, int lane) {
  uint32_t v = 0;
  if (NW >= 8) {
#pragma unroll
    for (int w = 0; w < NW; w += 8) v += (uint32_t)cnt[w * 8 + lane];
  } else {
    v = lane < NW * 8 ? (uint32_t)cnt[lane] : 0u;
  }
  v += dpp_move_u32<0x128>(v);  // row_ror:8
  u32x2_t r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  v = r[0] + r[1];
  r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return (int)(r[0] + r[1]);
}

struct Cut {
  uint32_t key;  // the k-th largest key
  int above;     // keys > key, or -1: exactly k keys are >= key (no ties to break)
};

// k-th largest of the keys key_of(it), it in [0, n_it), of all threads of NW waves; key 0 marks what does
// not take part, n_top < k keys are 0xFFFFFFFF.  With fewer than k others the result is key 0.  Must be reached
// by all NW waves (a workgroup's, if more than one); every thread gets the result.
template <int NW, int NT, int IPT, typename F>
__device__ __forceinline__ Cut kth_largest(F key_of, int n_it, int k, int n_top, SelectSmem<NW>& sm) {
  const int lane = threadIdx.x & 63, wave = NW == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const auto each = [&](auto f) {
    if constexpr (IPT > 0) {
#pragma unroll
      for (int it = 0; it < IPT; ++it)
        if (it < n_it) f(it);
    } else {
      for (int it = 0; it < n_it; ++it) f(it);
    }
  };
  // invariant: at least k keys are >= lo (`reach`, or fewer at first), fewer than k are >= hi, namely `above`
  uint32_t lo = 1u, hi = 0xFFFFFFFFu;
  int above = n_top, reach = 64 * NW * n_it;
  // closes lo and hi in on the keys between them; false: there are none
  const auto close_in = [&]() -> bool {
    uint32_t below = 0xFFFFFFFFu, behind = 0xFFFFFFFFu;  // room at the ends (keys outside wrap to at least hi - lo)
    each([&](int it) {
      const uint32_t key = key_of(it);
      below = min(below, key - lo);
      behind = min(behind, hi - 1u - key);
    });
    int mb = wave_max_i((int)(~below ^ 0x80000000u)), mh = wave_max_i((int)(~behind ^ 0x80000000u));
    if constexpr (NW > 1) {
      __syncthreads();  // the scratch arrays are free
      if (lane == 0) { sm.lo[wave] = mb; sm.hi[wave] = mh; }
      __syncthreads();
#pragma unroll
      for (int w = 0; w < NW; ++w) { mb = max(mb, sm.lo[w]); mh = max(mh, sm.hi[w]); }
    }
    below = (uint32_t)__builtin_amdgcn_readfirstlane(~(mb ^ (int)0x80000000u));
    behind = (uint32_t)__builtin_amdgcn_readfirstlane(~(mh ^ (int)0x80000000u));
    if (below >= hi - lo) return false;
    lo += below;
    hi -= behind;
    return true;
  };
  if (!close_in()) return {0u, n_top};  // nothing else takes part
  // (the smallest key itself is never counted: fewer than k keys in all end at lo with above < k)
  for (int round = 1; hi - lo > 1; ++round) {
    const uint32_t w = hi - lo;
    const uint32_t step = w > NT + 1 ? w / (NT + 1) : 1u;
    uint32_t c[NT];
    int n[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      c[i] = step * (i + 1) < w ? lo + step * (i + 1) : hi - 1;  // repeats of hi - 1 do no harm
      n[i] = 0;
    }
    each([&](int it) {
      const uint32_t key = key_of(it);
#pragma unroll
      for (int i = 0; i < NT; ++i) n[i] += __popcll(__ballot(key >= c[i]));
    });
    if constexpr (NW > 1) {
      int mine = 0;
#pragma unroll
      for (int i = 0; i < NT; ++i) mine = lane == i ? n[i] : mine;
      int* cnt = sm.cnt[round & 1];
      if (lane < 8) cnt[wave * 8 + lane] = mine;
      __syncthreads();
      const int sum = sum_counts<NW>(cnt, lane);
#pragma unroll
      for (int i = 0; i < NT; ++i) n[i] = __builtin_amdgcn_readlane(sum, i);
    }
    uint32_t new_lo = lo, new_hi = hi;
    const int inside = reach - above;
#pragma unroll
    for (int i = NT - 1; i >= 0; --i) {  // counts fall with i
      if (n[i] == k) return {c[i], -1};
      if (n[i] < k) { new_hi = c[i]; above = n[i]; }
      else if (c[i] > new_lo) { new_lo = c[i]; reach = n[i]; }
    }
    lo = new_lo;
    hi = new_hi;
    // a range that shrank and lost few of its keys is mostly empty (ties, outliers, clusters): the rest is left at
    // once.  (Not in the first round: scores fill the upper end of their range, an octave like the next.  Nor with
    // 32 keys per thread, whose registers are all taken.)
    if constexpr (IPT <= 16)
      if (round > 1 && 8 * (long long)(reach - above) > 7 * (long long)inside && hi - lo > 1) close_in();
  }
  return {lo, above};
}

// Row window and exponent slope of one head's forgotten score (Section 3.3 Eq.5): rows before
// `first_row` have a weight alpha^(n-1-i) below the smallest fp32 subnormal and add exactly 0.
// On entry first_row / log2_alpha are the host's values for its bound alpha_max (log2_alpha is 0
// for both alpha_max = 1, with first_row 0, and alpha_max = 0, with first_row n-1).  With
// alpha_heads the head's own factor narrows the window; a factor above the bound is computed
// as the bound.
__device__ __forceinline__ void head_window(const float* alpha_heads, int g, int n, int& first_row,
                                            float& log2_alpha) {
  if (!alpha_heads) return;  // host values apply to every head
  const float a = alpha_heads[g];
  if (!(a > 0.f)) { first_row = n - 1; log2_alpha = 0.f; return; }   // alpha = 0: the newest row only
  if (log2_alpha == 0.f && first_row >= n - 1) return;               // bound is 0 (or n = 1)
  float l2 = a < 1.f ? log2f(a) : 0.f;
  if (log2_alpha < 0.f) l2 = fminf(l2, log2_alpha);                  // bound below 1: clamp
  log2_alpha = l2;
  if (l2 == 0.f) return;                                             // alpha = 1 under a bound of 1: all rows
  const float rows = 160.0f / (-l2);
  const int own = rows >= (float)n ? 0 : n - ((int)rows + 1);
  first_row = own > first_row ? own : first_row;
}

__device__ __forceinline__ uint4 load16(const void* p) { return *reinterpret_cast<const uint4*>(p); }
// 16 bytes that are read once and not again soon (the streamed rows of a KV cache): the
// non-temporal hint keeps them from displacing other lines on their way through the caches.
// Measured on MI355X with reads of 1.7 GB: 7.0-7.1 TB/s with the hint, 6.2-6.3 TB/s without.
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 load16_stream(const void* p) {
  const u32x4_t v = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(p));
  return make_uint4(v.x, v.y, v.z, v.w);
}
template <bool STREAM>
__device__ __forceinline__ uint4 load16_as(const void* p) {
  return STREAM ? load16_stream(p) : load16(p);
}
// Direct global-to-LDS load: 16 (or 4) bytes at base + lane_off of every lane land at
// lds_addr + 16 (4) * lane.  base and lds_addr are the same for the whole wave.  Written as an
// instruction of its own and not through the compiler's builtin, because for the builtin the
// compiler waits for ALL outstanding direct loads before the next LDS read of the same array
// (it cannot tell the ring stages apart), which undoes every prefetch.  The loads are invisible
// to the compiler's wait counting: the kernel waits itself (wait_vm, wait_vm_barrier) before the data is
// read, and makes sure that a stage's readers are done before it is filled again.  The compiler's
// own waits stay correct, since loads return in order: it can only wait for more than it needs.
// The statements keep the distances themselves that the hardware does not: one state between the M0
// write and the load, and five between a vector instruction that writes a scalar register and a load that reads
// it -- the compiler may have formed the base with one (v_readfirstlane) right before, so the load reads a copy
// that a scalar move made.  M0 cannot be declared as clobbered: it is a reserved register, which the compiler
// keeps no value in across a statement but writes right before each of its own uses.
__device__ __forceinline__ void dma16(const void* base, uint32_t lane_off, uint32_t lds_addr) {
  const void* copy;
  asm volatile("s_mov_b32 m0, %1\n\ts_mov_b64 %0, %3\n\tglobal_load_lds_dwordx4 %2, %0"
               : "=&s"(copy) : "s"(__builtin_amdgcn_readfirstlane(lds_addr)), "v"(lane_off), "s"(base) : "memory");
}
// ... from an address per lane
__device__ __forceinline__ void dma16_at(const void* p, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
               :: "s"(__builtin_amdgcn_readfirstlane(lds_addr)), "v"(p) : "memory");
}
__device__ __forceinline__ void dma4(const void* base, uint32_t lane_off, uint32_t lds_addr) {
  const void* copy;
  asm volatile("s_mov_b32 m0, %1\n\ts_mov_b64 %0, %3\n\tglobal_load_lds_dword %2, %0"
               : "=&s"(copy) : "s"(__builtin_amdgcn_readfirstlane(lds_addr)), "v"(lane_off), "s"(base) : "memory");
}
// At most LEFT of this wave's loads and stores outstanding.  LDS reads are another matter: before a tile is filled again
// its readers need wait_lds too (or wait_vm_barrier, which waits for both).
template <int LEFT>
__device__ __forceinline__ void wait_vm() { asm volatile("s_waitcnt vmcnt(%0)" :: "n"(LEFT) : "memory"); }
__device__ __forceinline__ void wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
// Workgroup barrier that leaves LEFT of the wave's loads under way (a plain __syncthreads may
// wait for all of them); the wave's LDS accesses are done.
template <int LEFT>
__device__ __forceinline__ void wait_vm_barrier() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(LEFT) : "memory");
}
__device__ __forceinline__ void store16(void* p, const uint4& v) { *reinterpret_cast<uint4*>(p) = v; }

// Launch order of a kernel whose items are nb blocks of G heads, the heaviest block of a head (rank 0)
// down to the lightest.  The grid is dispatched in order, workgroups to the 8 accelerator dies in turn, so
// - a whole head belongs to one die, whose L2 its blocks share; heads that do not divide by 8 are dealt
//   out block by block;
// - a die's heads go through their ranks together: what is left for the end are the lightest blocks of all of
//   them, not one head's heavy ones (head after head / in this order: fp32 attention, 32 heads x 1000 rows 117 / 101 us,
//   4 x 3000 172 / 146; bf16 attention, d = 64, 96 x 1777 74 / 67, chunk of 512 x 512 rows 143 / 128);
// - but only so many heads at a time as fill the die about three times over: their keys have to stay in its L2.
__host__ __device__ inline int ordered_heads(int nb) {
  const int f = 192 / nb;
  return 8 * (f < 1 ? 1 : (f > 8 ? 8 : f));
}
inline unsigned ordered_grid(int G, int nb) {
  const int rest = G % ordered_heads(nb);
  return (unsigned)((long long)(G - rest) * nb + (long long)rest * (rest % 8 ? (nb + 7) / 8 * 8 : nb));
}
// This workgroup's head and rank; false: none.
__device__ __forceinline__ bool ordered_item(int G, int nb, int& head, int& rank) {
  const unsigned heads = (unsigned)ordered_heads(nb);
  const unsigned chunk = min(blockIdx.x / (heads * (unsigned)nb), (unsigned)G / heads);
  const unsigned here = min(heads, (unsigned)G - chunk * heads);  // heads of this chunk
  unsigned w = blockIdx.x - chunk * heads * (unsigned)nb;
  const unsigned full = here / 8, odd = here % 8;  // heads per die, heads dealt out
  const unsigned period = w / (8 * here);          // eight ranks of the chunk's heads
  w -= period * 8 * here;
  if (w < 64 * full) {
    rank = (int)(8 * period + w / (8 * full));
    head = (int)(chunk * heads + w % 8 * full + w / 8 % full);
  } else {
    w -= 64 * full;
    rank = (int)(8 * period + w / odd);
    head = (int)(chunk * heads + 8 * full + w % odd);
  }
  return rank < nb;
}

}  // namespace a2sf
