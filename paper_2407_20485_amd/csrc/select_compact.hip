// Per-head token selection (top-k with a protected recent window) and compaction of the
// KV cache.  Section 2.2 / Section 3.1 of the paper: the tokens with the smallest
// accumulated score leave the cache; Section 4.1: the budget has a score-selected and a
// most-recent part.  Ties go to the lower original position.
//
// Selection: one workgroup per head.  A head's scores become order-preserving integer keys, held in
// registers where they fit, and the cut (a key that exactly `select` tokens reach) is found by a
// search over the key range (kth_largest): every round counts the keys at or above three thresholds at
// once, one compare and one scalar bit count per wave, key and threshold, and keeps the
// subinterval that holds the cut.  It ends as soon as a threshold separates exactly `select`
// tokens, after six to nine rounds on real scores; where a subinterval keeps nearly all of its keys (ties, outliers,
// clusters) the bounds close in on them.  A histogram of digits (the usual radix
// select) sends most keys of a head to a few bins -- scores share their sign and most of
// their exponent -- where the LDS atomics serialise (us per call, that way / here: 32 heads x 32768 tokens 195 / 47,
// 32 x 1024 9.5 / 8.4, 2048 x 2048 27 / 24, the same with most scores 0 106 / 33, 8000 x 400 32 / 18).  Seven thresholds
// need fewer rounds and more work per bit (8000 x 200: 12.0 and 15.1).  Up to three searches run:
//   1. the `recent`-th largest position           -> who is in the recent window (only where the
//      newest positions have gaps; otherwise the largest position tells)
//   2. the `select`-th largest score of the rest  -> score threshold
//   3. among scores equal to the threshold, the position below which ties are kept
// followed by an ordered emission (prefix sum over the waves) of the surviving slot indices.
#include "a2sf_dev.h"
#include "a2sf_internal.h"
#include "select_dev.h"

namespace a2sf {
namespace {

// T threads per head.  SOLO: one of the waves does the search alone (up to 64 * IPT tokens, keys in registers), the others
// only take part in the copy.  Otherwise all waves do.
// MOVE: the kept indices stay in LDS (B <= kFusedKeep) and the workgroup moves the rows of its head at once.
// kGather: from a prompt into the cache (pos and len are null).  kInPlace: in the cache; a chunk's tokens (to.kin) are the
// last to.m, in front of them len[g] others.
template <int T, int IPT, bool SOLO, int MOVE>
__global__ __launch_bounds__(T) void select_kernel(
    const float* __restrict__ scores, const int32_t* __restrict__ pos, const int32_t* __restrict__ len, int L, int stride,
    int select, int recent, int32_t* __restrict__ keep_idx, int32_t* __restrict__ n_keep, MoveTo to) {
  constexpr int NW = SOLO ? 1 : T / 64;  // waves that search
  __shared__ SelectSmem<NW> sm;
  __shared__ int list[kFusedKeep];
  const int g = blockIdx.x, tid = threadIdx.x;
  const int wave = SOLO ? 0 : __builtin_amdgcn_readfirstlane(tid >> 6);
  const int B = select + recent;
  int Lg = MOVE == kInPlace ? to.len[g] : (len ? len[g] : L);
  int off = to.capacity;  // in place: slots from here on have their rows in the second source
  if constexpr (MOVE == kInPlace) {
    if (to.off_heads && to.off_heads[g] < 0) return;
    if (to.kin) {
      if (Lg < 0 || Lg > to.capacity - to.m) return;
      off = Lg;
      Lg += to.m;
    }
  }
  Lg = Lg < 0 ? 0 : (Lg > L ? L : Lg);
  // (in place the arrays change: they are not the restricted arguments)
  const float* sc = (MOVE == kInPlace ? to.s : scores) + (size_t)g * stride;
  const int32_t* ps = MOVE == kInPlace ? to.p + (size_t)g * stride : (pos ? pos + (size_t)g * stride : nullptr);
  int32_t* out = MOVE ? list : keep_idx + (size_t)g * B;
  const int kept = min(Lg, B);
  const auto score = [&](int j) { return sc[j]; };
  const auto position = [&](int j) { return ps[j]; };

  if (Lg <= B) {
    for (int j = tid; j < Lg; j += T) out[j] = j;
  } else if (!SOLO || T == 64 || __builtin_amdgcn_readfirstlane(tid >> 6) == (int)(blockIdx.x / 8) % (T / 64)) {
    select_slots<NW, IPT>(score, position, ps != nullptr, Lg, select, recent, wave, out, sm);
  }
  if constexpr (MOVE == kSelectOnly) {
    if (tid == 0) n_keep[g] = kept;
    return;
  }
  __syncthreads();
  if (tid == 0) to.len[g] = kept;
  if constexpr (MOVE == kInPlace) {
    if (kept == 0 || (list[kept - 1] == kept - 1 && kept <= off)) return;  // nothing moves (the list ascends)
    move_rows<T>(to, list, kept, g, off, false, score, position);
  } else {
    gather_rows<T>(to, list, kept, g, L, score);
  }
}

template <int MOVE>
void launch_select_kernel(const float* scores, const int32_t* pos, const int32_t* len, int G, int L,
                          int stride, int select, int recent, int32_t* keep_idx, int32_t* n_keep,
                          const MoveTo& to, hipStream_t st) {
#define A2SF_SELECT(T, IPT, SOLO)                                                                         \
  hipLaunchKernelGGL((select_kernel<T, IPT, SOLO, MOVE>), dim3(G), dim3(T), 0, st, scores, pos, len, L, stride, \
                     select, recent, keep_idx, n_keep, to)
  // A search by one wave has no barriers: short heads, and longer ones of which there are so many that the
  // work counts and not the chain of rounds (us, one wave / four: 300 heads x 200 5.6 / 6.4, 8000 x 400 18.5 / 35.5,
  // 8000 x 1000 34 / 48, but 1500 x 1024 16.7 / 14.3 and 300 x 1024 14.5 / 8.4).  Up to 2048 slots four waves, or eight where
  // every head's workgroup has a compute unit (2048 slots, four / eight: 32 heads 12.0 / 10.2, 1500 heads 20.2 / 25.1; 16 of
  // them: 12.3 and 58.7).  Copying workgroups have more waves while there are few heads.
  constexpr bool copies = MOVE != kSelectOnly;
  const bool few = G <= 512;
  if constexpr (copies) {
    if (L <= 256) {
      if (few) A2SF_SELECT(512, 4, true); else A2SF_SELECT(256, 4, true);
      return;
    }
  } else {
    if (L <= 256) { A2SF_SELECT(64, 4, true); return; }
    if (L <= 512 && !few) { A2SF_SELECT(64, 8, true); return; }
    if (L <= 1024 && G > 2048) { A2SF_SELECT(64, 16, true); return; }
  }
  if (L <= 1024 && !(copies && few)) A2SF_SELECT(256, 4, false);
  else if (L <= 2048 && !few) A2SF_SELECT(256, 8, false);
  else if (L <= 2048) A2SF_SELECT(512, 4, false);
  else if (L <= 4096) A2SF_SELECT(1024, 4, false);
  else if (L <= 8192) A2SF_SELECT(1024, 8, false);
  else if (L <= 16384) A2SF_SELECT(1024, 16, false);
  else if (L <= 32768) A2SF_SELECT(1024, 32, false);
  else A2SF_SELECT(1024, 0, false);
#undef A2SF_SELECT
}

// ---------------------------------------------------------------------------------------
// In-place stable compaction.  keep[] is strictly ascending, so destination r <= source
// keep[r].  Rows are processed in ascending chunks; inside a chunk every source row is in
// registers before (barrier) any destination row is written.  A later chunk's sources lie
// at or beyond its own destinations, i.e. beyond everything written so far.
// Second source (kin != null): the K/V rows of the slots from off_heads[g] on have not been
// stored in the cache yet; they are rows 0 .. m-1 of kin / vin [G, m, ...] (a chunk of a
// prompt).  Kept rows among them are copied in; they follow every kept cached row, so no
// cached row that is still to be moved lies at or behind their destinations.
//
// Columns do not meet, so a head's rows are cut into slices of 128 bytes that move independently:
// 2 * ROW_UNITS / kSliceUnits workgroups per head (K, V), slice 0 also moves scores and positions.  A
// workgroup then has 256 rows under way per round instead of 64, and few heads still fill the chip
// (a round is a round trip to memory and two barriers; 320 heads x 410 rows, nearly all of them
// moving: 48.6 us with one workgroup per head, 19.4 us here; 512 heads, 512 of 1024 rows kept: 100 and 57 us).
constexpr int kSliceUnits = 8;
template <int ROW_UNITS>  // 16-byte units per K (or V) row
__device__ __forceinline__ void move_slice(int g, int part, int nk, int off, uint4* K, uint4* V, float* S, int32_t* P,
                                           int capacity, const int32_t* keep, const uint4* kin, const uint4* vin, int m) {
  constexpr int U = 8;                            // rows per thread per round
  constexpr int RPT = kThreads / kSliceUnits;     // rows per pass of the workgroup
  constexpr int CH = RPT * U;                     // rows per round
  constexpr int SL = ROW_UNITS / kSliceUnits;     // slices per K (or V) row
  static_assert(CH == kThreads, "a round moves one score per thread");
  const int tid = threadIdx.x;
  const int col = (part % SL) * kSliceUnits + tid % kSliceUnits;
  u32x4_t* X = reinterpret_cast<u32x4_t*>(part < SL ? K : V) + (size_t)g * capacity * ROW_UNITS + col;
  const u32x4_t* in = kin ? reinterpret_cast<const u32x4_t*>(part < SL ? kin : vin) + (size_t)g * m * ROW_UNITS + col : nullptr;
  float* Sg = S + (size_t)g * capacity;
  int32_t* Pg = P + (size_t)g * capacity;
  for (int r0 = 0; r0 < nk; r0 += CH) {
    u32x4_t x[U];
    int src[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int r = r0 + u * RPT + tid / kSliceUnits;
      src[u] = r < nk ? keep[r] : r;
      src[u] = src[u] < 0 ? 0 : (src[u] >= capacity ? capacity - 1 : src[u]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int r = r0 + u * RPT + tid / kSliceUnits;
      if (r >= nk) src[u] = -1;
      else if (src[u] >= off) x[u] = in[(src[u] - off < m ? src[u] - off : m - 1) * ROW_UNITS];
      else if (src[u] != r) x[u] = X[src[u] * ROW_UNITS];
      else src[u] = -1;  // stays where it is
    }
    float s_val = 0.f;
    int p_val = 0;
    bool mv_s = false;
    if (part == 0 && r0 + tid < nk) {
      int from = keep[r0 + tid];
      from = from < 0 ? 0 : (from >= capacity ? capacity - 1 : from);
      if (from != r0 + tid) { mv_s = true; s_val = Sg[from]; p_val = Pg[from]; }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (src[u] >= 0) X[(r0 + u * RPT + tid / kSliceUnits) * ROW_UNITS] = x[u];
    if (mv_s) { Sg[r0 + tid] = s_val; Pg[r0 + tid] = p_val; }
  }
}

__device__ __forceinline__ int rows_kept(int nk, int capacity, int keep_stride) {
  nk = nk < 0 ? 0 : (nk > capacity ? capacity : nk);
  return nk > keep_stride ? keep_stride : nk;
}

template <int ROW_UNITS>
__global__ __launch_bounds__(kThreads) void compact_kernel(
    uint4* __restrict__ K, uint4* __restrict__ V, float* __restrict__ S, int32_t* __restrict__ P,
    int32_t* __restrict__ len, int capacity, const int32_t* __restrict__ keep_idx, int keep_stride,
    const int32_t* __restrict__ n_keep, const uint4* __restrict__ kin, const uint4* __restrict__ vin,
    int m, const int32_t* __restrict__ off_heads) {
  constexpr int PER = 2 * ROW_UNITS / kSliceUnits;  // workgroups per head
  const int g = blockIdx.x / PER, part = blockIdx.x % PER;
  const int nk = rows_kept(n_keep[g], capacity, keep_stride);
  if (off_heads && off_heads[g] < 0) return;      // a head the chunk did not fit into: untouched
  const int off = kin ? off_heads[g] : capacity;  // slots from here on live in the second source
  const int32_t* keep = keep_idx + (size_t)g * keep_stride;
  if (part == 0 && threadIdx.x == 0) len[g] = nk;  // (no other workgroup reads it)
  // strictly ascending indices: the identity if the last one is in its own slot
  if (nk == 0 || (keep[nk - 1] == nk - 1 && nk <= off)) return;
  move_slice<ROW_UNITS>(g, part, nk, off, K, V, S, P, capacity, keep, kin, vin, m);
}

// Where hardly a head has anything to move (the stable steps of many heads, whose kernel has moved the rows already):
// a workgroup looks at eight heads at once, one lane each, and moves its slice of those that do move, one after the other
// (16384 heads x 201 slots with nothing to move: 27 us with four workgroups per head, 7.2 here; 4096 fp32 heads x 101 x
// 128 that all move, because the newest positions have gaps: 147 us, 176 when one workgroup takes all slices of its eight).
constexpr int kSparseHeads = 8;
template <int ROW_UNITS>
__global__ __launch_bounds__(kThreads) void compact_sparse_kernel(
    uint4* __restrict__ K, uint4* __restrict__ V, float* __restrict__ S, int32_t* __restrict__ P,
    int32_t* __restrict__ len, int G, int capacity, const int32_t* __restrict__ keep_idx, int keep_stride,
    const int32_t* __restrict__ n_keep) {
  constexpr int PER = 2 * ROW_UNITS / kSliceUnits;  // workgroups per eight heads
  const int g0 = blockIdx.x / PER * kSparseHeads, part = blockIdx.x % PER, lane = threadIdx.x & 63;
  bool moves = false;
  if (lane < kSparseHeads && g0 + lane < G) {
    const int nk = rows_kept(n_keep[g0 + lane], capacity, keep_stride);
    if (part == 0 && threadIdx.x < kSparseHeads) len[g0 + lane] = nk;
    moves = nk > 0 && keep_idx[(size_t)(g0 + lane) * keep_stride + nk - 1] != nk - 1;
  }
  for (unsigned long long left = __ballot(moves); left; left &= left - 1) {  // (every wave has the same)
    const int g = g0 + __builtin_ctzll(left), nk = rows_kept(n_keep[g], capacity, keep_stride);
    move_slice<ROW_UNITS>(g, part, nk, capacity, K, V, S, P, capacity, keep_idx + (size_t)g * keep_stride, nullptr,
                          nullptr, 0);
  }
}

// Out-of-place gather of surviving prompt rows.  grid = G * chunks (head-major).
template <int ROW_UNITS>
__global__ __launch_bounds__(kThreads) void gather_prompt_kernel(
    const uint4* __restrict__ Kin, const uint4* __restrict__ Vin, const float* __restrict__ Sfull,
    int n, const int32_t* __restrict__ keep_idx, int keep_stride, const int32_t* __restrict__ n_keep,
    uint4* __restrict__ K, uint4* __restrict__ V, float* __restrict__ S, int32_t* __restrict__ P,
    int32_t* __restrict__ len, int capacity, int chunks) {
  constexpr int ROWS = kThreads / ROW_UNITS;
  const int g = blockIdx.x / chunks, chunk = blockIdx.x % chunks, tid = threadIdx.x;
  const int nk = n_keep[g];
  const int r = chunk * ROWS + tid / ROW_UNITS, c = tid % ROW_UNITS;
  if (chunk == 0 && tid == 0) len[g] = nk;
  if (r >= nk || r >= capacity || r >= keep_stride) return;
  int src = keep_idx[(size_t)g * keep_stride + r];
  src = src < 0 ? 0 : (src >= n ? n - 1 : src);
  const size_t in = ((size_t)g * n + src) * ROW_UNITS + c;
  const size_t out = ((size_t)g * capacity + r) * ROW_UNITS + c;
  K[out] = Kin[in];
  V[out] = Vin[in];
  if (c == 0) {
    S[(size_t)g * capacity + r] = Sfull[(size_t)g * n + src];
    P[(size_t)g * capacity + r] = src;
  }
}

inline int row_units(int d, int dtype) { return d * (dtype == A2SF_BF16 ? 2 : 4) / 16; }

}  // namespace

void launch_select(const float* scores, const int32_t* pos, const int32_t* len, int G, int L,
                   int stride, int select, int recent, int32_t* keep_idx, int32_t* n_keep,
                   hipStream_t st) {
  launch_select_kernel<kSelectOnly>(scores, pos, len, G, L, stride, select, recent, keep_idx, n_keep, MoveTo{}, st);
}

void launch_compact(const a2sf_cache& c, const int32_t* keep_idx, int keep_stride,
                    const int32_t* n_keep, hipStream_t st, const void* k2, const void* v2, int m2,
                    const int32_t* off_heads, bool mostly_done) {
  const int ru = row_units(c.d, c.dtype);
#define A2SF_COMPACT(RU)                                                                        \
  do {                                                                                          \
    if (mostly_done)                                                                            \
      hipLaunchKernelGGL(compact_sparse_kernel<RU>, dim3((unsigned)(c.G + kSparseHeads - 1) / kSparseHeads * (2 * RU / kSliceUnits)), \
                         dim3(kThreads), 0, st, (uint4*)c.k, (uint4*)c.v, c.scores, c.pos, c.len, c.G,      \
                         c.capacity, keep_idx, keep_stride, n_keep);                            \
    else                                                                                        \
      hipLaunchKernelGGL(compact_kernel<RU>, dim3((unsigned)c.G * (2 * RU / kSliceUnits)), dim3(kThreads), 0, st, \
                         (uint4*)c.k, (uint4*)c.v, c.scores, c.pos, c.len, c.capacity, keep_idx, keep_stride, \
                         n_keep, (const uint4*)k2, (const uint4*)v2, m2, off_heads);            \
  } while (0)
  if (ru == 8) A2SF_COMPACT(8);
  else if (ru == 16) A2SF_COMPACT(16);
  else A2SF_COMPACT(32);
#undef A2SF_COMPACT
}

// One workgroup moves a head's rows, up to 128 KB of K: a launch and a round trip through the index list less (us per call,
// two kernels / this one, bf16, d = 128: chunk of 111 rows, 3 heads keeping 45, 25.4 / 21.2; 512 heads keeping 512,
// 230 / 221; stable step of 243 heads x 8 queries, 174 slots, 34.4 / 28.6; 4 x 4, 500 slots, 23.2 / 22.6).  More is moved
// sooner by a workgroup per slice (fp32, 500 slots, 256 KB: 30 heads 28 / 35, 600 heads 136 / 151), and with many heads the
// launch does not count (stable step of 3000 x 4, 500 slots, 351 / 355; fp32 chunk of 30 rows, 2000 heads, 226 / 229) unless
// `appends`, the kernel that would append the chunk is saved with it (2048 heads, 40 rows, 410 / 402).
constexpr int kInPlaceHeads = 1024;
bool selects_in_place(const a2sf_cache& c, int select, int recent, bool appends) {
  return select + recent <= kFusedKeep && (select + recent) * row_units(c.d, c.dtype) <= 8192 &&
         (appends || c.G <= kInPlaceHeads);
}

void launch_select_compact(const a2sf_cache& c, int select, int recent, hipStream_t st, const void* k2, const void* v2,
                           int m2, const int32_t* off_heads) {
  const MoveTo to = {(const u32x4_t*)k2, (const u32x4_t*)v2, (u32x4_t*)c.k, (u32x4_t*)c.v, c.scores, c.pos, c.len,
                     c.capacity, lg_row_units(row_units(c.d, c.dtype)), m2, off_heads};
  launch_select_kernel<kInPlace>(nullptr, nullptr, nullptr, c.G, c.capacity, c.capacity, select, recent, nullptr, nullptr,
                                 to, st);
}

void launch_select_gather(const void* k, const void* v, const float* scores_full, int n, int select,
                          int recent, int32_t* keep_idx, int32_t* n_keep, const a2sf_cache& c,
                          hipStream_t st) {
  const int ru = row_units(c.d, c.dtype);
  const int keep_stride = select + recent;
  // Short lists: the workgroup that selects also copies (up to 512 KB per head) -- one launch and one round
  // trip through the index list less.  Kernel times in two / in one, bf16: 2048 heads keeping 200 of 2048 rows,
  // d = 128, 95 / 84 us; 96 heads keeping 355 of 1777, d = 64, 15.0 / 12.3; 32 heads keeping 204 of 1024, d = 128,
  // 11.2 / 11.1.  A longer list is copied by more workgroups than one per head: 32 heads keeping 3276 of 32768
  // rows move 3.4 MB per head, 21 us with 205 workgroups per head.
  if (keep_stride <= kFusedKeep) {
    const MoveTo to = {(const u32x4_t*)k, (const u32x4_t*)v, (u32x4_t*)c.k, (u32x4_t*)c.v, c.scores, c.pos,
                       c.len, c.capacity, lg_row_units(ru), 0, nullptr};
    launch_select_kernel<kGather>(scores_full, nullptr, nullptr, c.G, n, n, select, recent, nullptr, nullptr, to, st);
    return;
  }
  launch_select(scores_full, nullptr, nullptr, c.G, n, n, select, recent, keep_idx, n_keep, st);
  const int rows = kThreads / ru;
  const int max_rows = keep_stride < c.capacity ? keep_stride : c.capacity;
  const int chunks = (max_rows + rows - 1) / rows;
  dim3 grid((unsigned)chunks * (unsigned)c.G);
#define A2SF_GATHER(RU)                                                                          \
  hipLaunchKernelGGL(gather_prompt_kernel<RU>, grid, dim3(kThreads), 0, st, (const uint4*)k,     \
                     (const uint4*)v, scores_full, n, keep_idx, keep_stride, n_keep, (uint4*)c.k, \
                     (uint4*)c.v, c.scores, c.pos, c.len, c.capacity, chunks)
  if (ru == 8) A2SF_GATHER(8);
  else if (ru == 16) A2SF_GATHER(16);
  else A2SF_GATHER(32);
#undef A2SF_GATHER
}

}  // namespace a2sf
