// Device side of the selection (see select_compact.hip): the search with its ordered emission, and the moves of the kept rows
// by the workgroup that has selected them.
#pragma once
#include "a2sf_dev.h"

namespace a2sf {

constexpr int kSelectOnly = 0, kGather = 1, kInPlace = 2;  // what a selection does with the kept rows

// Where the kept rows go, for kernels that select and move them.
constexpr int kFusedKeep = 512;  // tokens kept per head, at most
struct MoveTo {
  const u32x4_t *kin, *vin;  // a prompt's rows [G, L, row]; a chunk's [G, m, row], or null
  u32x4_t *k, *v;            // [G, capacity, row]
  float* s;
  int32_t *p, *len;
  int capacity, lg_units;    // log2 of the 16-byte units per row
  int m;                     // in place: tokens of the chunk
  const int32_t* off_heads;  // in place, may be null: negative entries mark heads to be left alone
};

inline int lg_row_units(int ru) { return ru == 8 ? 3 : (ru == 16 ? 4 : 5); }

// The indices of the surviving tokens of a head with Lg > select + recent tokens, ascending, to out; by all threads of
// NW waves (this one is `wave`).  score(j): a token's score; pos(j): its position if has_pos (otherwise that is j).
// IPT > 0: keys in registers, up to 64 * NW * IPT tokens; IPT = 0: any number, the keys formed again in every round.
template <int NW, int IPT, typename ScoreFn, typename PosFn>
__device__ __forceinline__ void select_slots(ScoreFn score, PosFn pos, bool has_pos, int Lg, int select, int recent, int wave,
                                             int32_t* out, SelectSmem<NW>& sm) {
  constexpr int NR = IPT > 0 ? IPT : 1;
  constexpr int NT = 3;  // thresholds per round
  const int lane = threadIdx.x & 63, B = select + recent;
  // a wave has 64 * n_it consecutive slots, iteration it its slots j0 + 64 it
  const int n_it = (Lg + NW * 64 - 1) / (NW * 64);
  const int j0 = wave * 64 * n_it + lane;
  const auto each = [&](auto f) {
    if constexpr (IPT > 0) {
#pragma unroll
      for (int it = 0; it < IPT; ++it)
        if (it < n_it) f(it, j0 + 64 * it);
    } else {
      for (int it = 0; it < n_it; ++it) f(it, j0 + 64 * it);
    }
  };
  uint32_t key[NR];
  if constexpr (IPT > 0)  // requested first
    each([&](int it, int j) { key[it] = __float_as_uint(score(j < Lg ? j : 0)); });

  // 1. recent window: positions >= p_recent
  uint32_t p[NR];  // position + 1, or 0
  const auto pos_key = [&](int it) -> uint32_t {
    if constexpr (IPT > 0) return p[it];
    else { const int j = j0 + 64 * it; return j < Lg ? (uint32_t)pos(j) + 1u : 0u; }
  };
  int p_recent = 0;
  if (recent > 0) {
    if (!has_pos) {
      p_recent = Lg - recent;
    } else {
      if constexpr (IPT > 0) each([&](int it, int j) { p[it] = j < Lg ? (uint32_t)pos(j) + 1u : 0u; });
      // a cache that always kept its newest tokens holds exactly `recent` positions > newest - recent
      uint32_t newest = 0;
      int cnt = 0;
      each([&](int it, int) { newest = max(newest, pos_key(it)); });
      int most = wave_max_i((int)(newest ^ 0x80000000u));
      if constexpr (NW > 1) {
        if (lane == 0) sm.hi[wave] = most;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < NW; ++w) most = max(most, sm.hi[w]);
      }
      newest = (uint32_t)__builtin_amdgcn_readfirstlane(most) ^ 0x80000000u;
      each([&](int it, int) { cnt += __popcll(__ballot(pos_key(it) > newest - (uint32_t)recent)); });
      if constexpr (NW > 1) {
        if (lane < 8) sm.cnt[0][wave * 8 + lane] = cnt;
        __syncthreads();
        cnt = __builtin_amdgcn_readfirstlane(sum_counts<NW>(sm.cnt[0], lane));
      }
      if (cnt == recent) p_recent = (int)(newest - (uint32_t)recent);  // (newest is a position + 1)
      else p_recent = (int)(kth_largest<NW, NT, IPT>(pos_key, n_it, recent, 0, sm).key - 1u);
    }
  }
  // 2. score threshold.  Keys: 0 past the end, all ones in the recent window (which is always
  // kept, so that the cut is simply the B-th largest key), the ordered score of the others.
  const auto form_key = [&](int it, int j, uint32_t bits) -> uint32_t {
    const bool r = recent > 0 && (has_pos ? pos_key(it) > (uint32_t)p_recent : j >= p_recent);
    return j < Lg ? (r ? 0xFFFFFFFFu : score_key(__uint_as_float(bits))) : 0u;
  };
  if constexpr (IPT > 0) each([&](int it, int j) { key[it] = form_key(it, j, key[it]); });
  const auto key_of = [&](int it) -> uint32_t {
    if constexpr (IPT > 0) return key[it];
    else { const int j = j0 + 64 * it; return form_key(it, j, __float_as_uint(score(j < Lg ? j : 0))); }
  };
  Cut cut = {0xFFFFFFFFu, -1};
  if (select > 0) cut = kth_largest<NW, NT, IPT>(key_of, n_it, B, recent, sm);
  // 3. ties at the cut: the lowest positions stay
  uint32_t tie_cut = 0u;  // they have 2^31 - position >= tie_cut
  const auto tie_key = [&](int it) -> uint32_t {
    const int j = j0 + 64 * it;
    return j < Lg && key_of(it) == cut.key ? 0x80000000u - (uint32_t)(has_pos ? pos(j) : j) : 0u;
  };
  if (cut.above >= 0) tie_cut = kth_largest<NW, NT, IPT>(tie_key, n_it, B - cut.above, 0, sm).key;

  // 4. ordered emission
  const auto keeps = [&](int it) -> bool {
    const uint32_t k = key_of(it);
    if (cut.above < 0) return k >= cut.key;
    return k > cut.key || (k == cut.key && tie_key(it) >= tie_cut && tie_cut != 0u);
  };
  int base = 0;
  if constexpr (NW > 1) {
    int total = 0;
    each([&](int it, int) { total += __popcll(__ballot(keeps(it))); });
    __syncthreads();
    if (lane == 0) sm.lo[wave] = total;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < NW; ++w) base += w < wave ? sm.lo[w] : 0;
    base = __builtin_amdgcn_readfirstlane(base);
  }
  each([&](int it, int j) {
    const bool k = keeps(it);
    const unsigned long long mask = __ballot(k);
    const int at = base + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
    if (k && at < B) out[at] = j;  // bound holds for valid input; guards bad input
    base += __popcll(mask);
  });
}

// The kept rows of a prompt, by T threads: K, V in 16-byte units, four rows' units of each under way per thread.
template <int T, typename ScoreFn>
__device__ __forceinline__ void gather_rows(const MoveTo& to, const int32_t* list, int kept, int g, int L, ScoreFn score) {
  const int tid = threadIdx.x;
  const int units = kept << to.lg_units, mask = (1 << to.lg_units) - 1;
  const size_t in0 = ((size_t)g * L) << to.lg_units, out0 = ((size_t)g * to.capacity) << to.lg_units;
  for (int u0 = tid; u0 < units; u0 += 4 * T) {
    u32x4_t kx[4], vx[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int u = u0 + i * T;
      if (u < units) {
        const int src = min(max(list[u >> to.lg_units], 0), L - 1);
        const size_t at = in0 + (((size_t)src) << to.lg_units) + (u & mask);
        kx[i] = to.kin[at];
        vx[i] = to.vin[at];
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int u = u0 + i * T;
      if (u < units) { to.k[out0 + u] = kx[i]; to.v[out0 + u] = vx[i]; }
    }
  }
  for (int r = tid; r < kept; r += T) {
    const int src = min(max(list[r], 0), L - 1);
    to.s[(size_t)g * to.capacity + r] = score(src);
    to.p[(size_t)g * to.capacity + r] = src;
  }
}

// The kept rows of a cache, in place, by T threads; rows may move in ascending order as in move_slice.  Slots from `off` on
// have their rows in the second source.  score(j): a kept token's score; all of them are stored if `rescored`, otherwise those of
// the rows that move.  pos(j): its position.
template <int T, typename ScoreFn, typename PosFn>
__device__ __forceinline__ void move_rows(const MoveTo& to, const int32_t* list, int kept, int g, int off, bool rescored,
                                          ScoreFn score, PosFn pos) {
  const int tid = threadIdx.x;
  constexpr int U = 4;  // units of K and of V per thread and round
  const int lg = to.lg_units, rows = U * T >> lg;
  u32x4_t* const Kg = to.k + (((size_t)g * to.capacity) << lg);
  u32x4_t* const Vg = to.v + (((size_t)g * to.capacity) << lg);
  const u32x4_t* const kin = to.kin + (((size_t)g * to.m) << lg);
  const u32x4_t* const vin = to.vin + (((size_t)g * to.m) << lg);
  float* const Sg = to.s + (size_t)g * to.capacity;
  int32_t* const Pg = to.p + (size_t)g * to.capacity;
  for (int r0 = 0; r0 < kept; r0 += rows) {
    u32x4_t kx[U], vx[U];
    bool moves[U];
#pragma unroll
    for (int i = 0; i < U; ++i) {
      const int u = tid + i * T, r = r0 + (u >> lg), c = u & ((1 << lg) - 1);
      const int src = r < kept ? min(max(list[r], 0), to.capacity - 1) : r;
      moves[i] = r < kept && (src != r || src >= off);
      if (moves[i]) {
        const int at = (src >= off ? min(src - off, to.m - 1) : src) << lg | c;
        kx[i] = src >= off ? kin[at] : Kg[at];
        vx[i] = src >= off ? vin[at] : Vg[at];
      }
    }
    float s_val = 0.f;
    int p_val = 0, dst = -1;
    if (tid < rows && r0 + tid < kept) {
      const int src = min(max(list[r0 + tid], 0), to.capacity - 1);
      if (rescored || src != r0 + tid) { dst = r0 + tid; s_val = score(src); p_val = pos(src); }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < U; ++i) {
      const int u = tid + i * T;
      if (moves[i]) { Kg[(r0 << lg) + u] = kx[i]; Vg[(r0 << lg) + u] = vx[i]; }
    }
    if (dst >= 0) { Sg[dst] = s_val; Pg[dst] = p_val; }
  }
}

}  // namespace a2sf
