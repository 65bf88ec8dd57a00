// Score smoothing + per-head top-k (MaskKV Section 3.3: S_keep = argtopk(I, k_{l,h})), and the head-level
// budget formula of Stage 2.
//
// Prompts of up to 16384 positions: one workgroup per head pools the scores into registers (order-preserving
// 32-bit keys, up to 16 a thread), finds the exact cut and emits the positions in ascending order: one kernel.
// Longer prompts take two stages, because the keys of a head no longer fit a workgroup's registers:
//   chunk stage  one workgroup per 4096 prompt positions of a head: pools the scores and writes, in ascending
//                position order, every (key, position) whose key is at least t0, a lower bound of the k-th
//                largest key of the chunk (k = the head's budget).  The head's k-th largest key is never below a
//                chunk's k-th largest key (fewer than k keys of the whole head are above it), so every member of
//                the answer and all its ties are among the candidates.
//   final stage  one workgroup per head: exact selection over the candidates.
//
// What bounds all of this is latency, not bandwidth: the scores of 32 heads are 4 MB at most, and each kernel is a chain
// of load, reduction, histogram, scan and ordered write with a barrier between each two.  So the chain is kept short:
//   - range refinement: the key range [lo, hi] is cut into two bins per thread, an LDS histogram and one scan by
//     all threads locate the bin that holds the k-th largest key; that bin becomes the range.
//   - as soon as the bin holds at most 64 entries (after the first round, for scores without many ties) they are
//     listed and ranked against each other by one wave, larger key first, ties to the lower position.  That gives
//     a cut (key, position) and an entry is kept iff it does not come after the cut: ties need no further pass.
//   - a bin that is a single key with more entries than that is refined over the positions in the same way.
#include "kernels.hpp"

namespace maskkv {

namespace {

constexpr int kSelThreads = 1024;
constexpr int kSelWaves = kSelThreads / 64;
constexpr int kChunk = 4096;       // prompt positions per chunk-stage workgroup
constexpr int kSelLdsCap = 32768;  // final stage: candidates (keys, then positions) kept in LDS: 128 KB
constexpr int kRankable = 64;      // entries that one wave ranks against each other
constexpr int kMaxChunks = 1024;   // chunk offsets of a head are kept in LDS: prompts of up to 4 Mi tokens
// Prompts that one workgroup selects alone.
constexpr int kSinglePrompt = 16 * kSelThreads;

struct SelectParams {
  Lens lens;
  int H, BH, P_max, max_chunks;
  const float* scores;
  int64_t score_stride;
  int window, mode;
  const int32_t* budgets;
  int32_t* idx;
  int32_t* cu;
  int64_t capacity;
  uint32_t* cand_key;  // [BH][max_chunks][kChunk] candidates of the chunk stage
  int32_t* cand_pos;   // [BH][max_chunks][kChunk]
  int32_t* cand_cnt;   // [BH][max_chunks] candidates per chunk
};

__device__ __forceinline__ void fetch_select_arguments() {
  typedef SelectParams A;
  fetch_arguments({MASKKV_ARGUMENT(A, lens), MASKKV_ARGUMENT(A, H), MASKKV_ARGUMENT(A, capacity)});
}

__device__ __forceinline__ uint32_t order_key(float v) {
  uint32_t u = __builtin_bit_cast(uint32_t, v);
  if (u == 0x80000000u) u = 0u;                         // -0 and +0 compare equal: one key for both
  return u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);  // larger float <=> larger unsigned key
}
// Wave-level scans and reductions on the data-parallel-primitive path of the vector ALU (row shifts inside the
// rows of 16 lanes, then the two row broadcasts): six dependent vector instructions, no LDS round trips.
template <typename Op>
__device__ __forceinline__ int wave_scan(int v, int identity, Op op) {
  v = op(v, __builtin_amdgcn_update_dpp(identity, v, 0x111, 0xf, 0xf, false));  // row_shr:1
  v = op(v, __builtin_amdgcn_update_dpp(identity, v, 0x112, 0xf, 0xf, false));  // row_shr:2
  v = op(v, __builtin_amdgcn_update_dpp(identity, v, 0x114, 0xf, 0xf, false));  // row_shr:4
  v = op(v, __builtin_amdgcn_update_dpp(identity, v, 0x118, 0xf, 0xf, false));  // row_shr:8
  v = op(v, __builtin_amdgcn_update_dpp(identity, v, 0x142, 0xa, 0xf, false));  // row_bcast:15 into rows 1, 3
  v = op(v, __builtin_amdgcn_update_dpp(identity, v, 0x143, 0xc, 0xf, false));  // row_bcast:31 into rows 2, 3
  return v;
}

__device__ __forceinline__ int wave_incl_scan(int v) {
  return wave_scan(v, 0, [](int a, int b) { return a + b; });
}
__device__ __forceinline__ uint32_t wave_min(uint32_t v) {
  const int r = wave_scan((int)v, -1, [](int a, int b) { return (int)min((uint32_t)a, (uint32_t)b); });
  return (uint32_t)__builtin_amdgcn_readlane(r, 63);
}
__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
  const int r = wave_scan((int)v, 0, [](int a, int b) { return (int)max((uint32_t)a, (uint32_t)b); });
  return (uint32_t)__builtin_amdgcn_readlane(r, 63);
}

// Entries in the order of the answer: larger key first, ties to the lower position.
__device__ __forceinline__ uint64_t code_of(uint32_t key, uint32_t pos) { return (uint64_t)key << 32 | (uint32_t)~pos; }

template <int THREADS>
struct SelShared {
  static constexpr int kWaves = THREADS / 64;
  static constexpr int kBins = 2 * THREADS;
  int hist[kBins];
  uint32_t wmin[kWaves], wmax[kWaves];
  int wtot[kWaves], wbase[kWaves], wsum[2][kWaves];
  uint64_t list[kRankable];
  int listed;
  uint32_t lo, hi;
  int krem, pop;
  uint64_t cut;
};

template <int THREADS>
__device__ __forceinline__ void sel_clear(SelShared<THREADS>& s) {
  reinterpret_cast<u32x2*>(s.hist)[threadIdx.x] = u32x2{0u, 0u};
  if (threadIdx.x == 0) s.listed = 0;
}

// The current range [lo, hi] of values, the rank wanted inside it (from the largest) and how many entries it holds.
struct Range {
  uint32_t lo, hi;
  int krem, pop;
};

// Narrow `g` until it holds at most `enough` entries or a single value.  `each(f)` calls f(value, valid) for the entries of
// this thread; those that are not valid are `absent` or less, and LONG: a thread has so many that a test of each is worth a branch.
// All threads call this; the histogram is clear on entry and on return.
template <bool LONG, int THREADS, typename Each>
__device__ __forceinline__ void refine(SelShared<THREADS>& s, Range& g, int enough, uint32_t absent, Each&& each) {
  constexpr int kBins = SelShared<THREADS>::kBins;
  constexpr int kWaves = SelShared<THREADS>::kWaves;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  while (g.lo != g.hi && g.pop > enough) {
    const uint32_t width = g.hi - g.lo;
    const int shift = max(0, 32 - __clz(width) - (31 - __builtin_clz(kBins)));  // (width >> shift) < kBins
    // bins are counted from the top of the range: bin 0 holds the largest values
    if (LONG && g.lo > absent)
      each([&](uint32_t v, bool) {
        const uint32_t below = g.hi - v;
        if (below <= width) atomicAdd(&s.hist[below >> shift], 1);
      });
    else
      each([&](uint32_t v, bool valid) {
        const uint32_t below = g.hi - v;
        if (valid & (below <= width)) atomicAdd(&s.hist[below >> shift], 1);
      });
    __syncthreads();
    const u32x2 two = reinterpret_cast<u32x2*>(s.hist)[tid];
    reinterpret_cast<u32x2*>(s.hist)[tid] = u32x2{0u, 0u};
    const int h0 = (int)two[0], h1 = (int)two[1];
    const int incl = wave_incl_scan(h0 + h1);
    if (lane == 63) s.wtot[wave] = incl;
    __syncthreads();
    int above = incl - (h0 + h1);
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const int t = s.wtot[w];
      above += w < wave ? t : 0;
    }
    if (above < g.krem && above + h0 + h1 >= g.krem) {  // exactly one thread owns the bin
      const bool second = above + h0 < g.krem;
      const int bin = 2 * tid + (second ? 1 : 0);
      const uint32_t from = (uint32_t)bin << shift;  // (below g.hi, and not more than width)
      s.hi = g.hi - from;
      s.lo = g.hi - min(from + ((1u << shift) - 1u), width);
      s.krem = g.krem - above - (second ? h0 : 0);
      s.pop = second ? h1 : h0;
    }
    __syncthreads();
    g = Range{s.lo, s.hi, s.krem, s.pop};
  }
}

// The largest values of a thread's quad or row of 16 lanes, of which the lowest of a workgroup bounds the k-th largest from below where
// there are k quads or rows of them.
__device__ __forceinline__ uint32_t quad_max(uint32_t v) {
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xf, 0xf, false));         // quad_perm:[1,0,3,2]
  return max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xf, 0xf, false));      // quad_perm:[2,3,0,1]
}
__device__ __forceinline__ uint32_t row_max(uint32_t v) {
  v = quad_max(v);
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x124, 0xf, 0xf, false));        // row_ror:4
  return max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xf, 0xf, false));     // row_ror:8
}

// Key range of the workgroup's entries from every thread's own (one barrier).
template <int THREADS>
__device__ __forceinline__ void key_range(SelShared<THREADS>& s, uint32_t kmin, uint32_t kmax, uint32_t& lo, uint32_t& hi) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  kmin = wave_min(kmin);
  kmax = wave_max(kmax);
  if (lane == 0) {
    s.wmin[wave] = kmin;
    s.wmax[wave] = kmax;
  }
  __syncthreads();
  lo = s.wmin[0];
  hi = s.wmax[0];
#pragma unroll
  for (int w = 1; w < SelShared<THREADS>::kWaves; ++w) {
    lo = min(lo, s.wmin[w]);
    hi = max(hi, s.wmax[w]);
  }
}

// The code of the k-th entry in the order of the answer, or one that separates the first k from the rest (1 <= k <= n);
// `each(f)` calls f(key, position, valid) for the entries of this thread.
template <bool LONG, int THREADS, typename Each>
__device__ __forceinline__ uint64_t exact_cut(SelShared<THREADS>& s, uint32_t lo, uint32_t hi, int k, int n, uint32_t last_pos,
                                              Each&& each) {
  Range g{lo, hi, k, n};
  refine<LONG>(s, g, kRankable, 0u, [&](auto&& f) { each([&](uint32_t key, uint32_t, bool valid) { f(key, valid); }); });
  if (g.krem == g.pop) return code_of(g.lo, last_pos);  // the whole bin is kept
  const uint32_t key_from = g.lo, key_span = g.hi - g.lo;
  uint32_t last = 0xFFFFFFFFu, first = 0u;  // ~position
  if (g.pop > kRankable) {  // one key, many entries: refine over their positions (lowest first: ~position descending)
    const uint32_t tau = g.lo;
    g.lo = ~last_pos;
    g.hi = 0xFFFFFFFFu;
    refine<false>(s, g, kRankable, 0xFFFFFFFFu,
                  [&](auto&& f) { each([&](uint32_t key, uint32_t pos, bool valid) { f(~pos, valid && key == tau); }); });
    if (g.krem == g.pop) return (uint64_t)tau << 32 | g.lo;
    first = g.lo;
    last = g.hi;
  }
  const bool any = key_from > 0u && first == 0u && last == 0xFFFFFFFFu;  // (positions past the prompt have the key 0)
  if (LONG && any)
    each([&](uint32_t key, uint32_t pos, bool) {
      if (key - key_from <= key_span) s.list[atomicAdd(&s.listed, 1)] = code_of(key, pos);  // (g.pop <= kRankable of them)
    });
  else
    each([&](uint32_t key, uint32_t pos, bool valid) {
      if (valid & (key - key_from <= key_span) & (~pos >= first) & (~pos <= last)) s.list[atomicAdd(&s.listed, 1)] = code_of(key, pos);
    });
  __syncthreads();
  if (threadIdx.x < 64) {
    const uint64_t mine = (int)threadIdx.x < g.pop ? s.list[threadIdx.x] : 0u;
    int better = 0;
    for (int i = 0; i < g.pop; ++i) better += s.list[i] > mine ? 1 : 0;
    if ((int)threadIdx.x < g.pop && better == g.krem - 1) s.cut = mine;  // (codes are distinct)
  }
  __syncthreads();
  return s.cut;
}

// Pooled score of position j of a head (mean: in-range terms added from the lowest index upwards in fp32, one
// division by their count; max: the maximum), as an order-preserving key.
__device__ __forceinline__ uint32_t pooled_key(const float* x, int j, int P, int r, int mode) {
  const int lo = max(0, j - r);
  const int hi = min(P - 1, j + r);
  float v = x[lo];
  if (mode == MASKKV_POOL_MAX) {
    for (int t = lo + 1; t <= hi; ++t) v = fmaxf(v, x[t]);
  } else {
    for (int t = lo + 1; t <= hi; ++t) v = __fadd_rn(v, x[t]);
    v = __fdiv_rn(v, (float)(hi - lo + 1));
  }
  return order_key(v);
}

// x / w for a whole w of 1 .. 17, correctly rounded, given y = 1 / w correctly rounded: Markstein's correction of the product by its
// exact remainder (the result equals the quotient for every significand of x and each of these w).  Three instructions instead of a
// dozen; x has to be far from both ends of the exponents' range, so that neither step leaves it.
__device__ __forceinline__ float divided(float x, float w, float y) {
  const float q = x * y;
  return fmaf(fmaf(-q, w, x), y, q);
}
// 1 / w for these w, correctly rounded: one Newton step from within a last place of it.
__device__ __forceinline__ float inverse(float w) {
  const float y = __builtin_amdgcn_rcpf(w);
  return fmaf(fmaf(-w, y, 1.f), y, y);
}
constexpr uint32_t kDividableFrom = 67u << 23, kDividableTo = 187u << 23;  // bits of 2^-60 and 2^60

// The four positions from p0 (a multiple of 4) of a head, as loaded from min(max(p0, 0), P - 4): those outside the prompt take
// the neutral element.
__device__ __forceinline__ void within_prompt(float (&w)[4], int p0, int P, float neutral) {
  const int late = p0 - (P - 4);  // the load was moved down by so many
  if (p0 < 0 || late > 0) {
    const bool none = p0 < 0 || late >= 4, one = late & 1, two = late & 2;
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = one ? (e < 3 ? w[e < 3 ? e + 1 : 0] : neutral) : w[e];
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = two ? (e < 2 ? w[e < 2 ? e + 2 : 0] : neutral) : w[e];
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = none ? neutral : w[e];
  }
}

// Keys of G groups of four consecutive positions, group i at j0 + i * step, adjacent lanes adjacent groups (0 for positions past
// the prompt).  Every lane loads its own four positions; the others of its windows come from the lanes beside it, and only the
// first and the last lane load theirs (R rounded up to a piece of four) from memory.  All loads are under way before the first
// use, and positions outside the prompt take the neutral element of the pooling, which leaves the sum (resp. the maximum) of the
// in-range terms as it is.
// R: radius of the window, or (not FIXED) a bound of it.  P >= 4, j0 and step multiples of 4, all lanes of a wave together.
template <int R, bool FIXED, int MODE, int G>
__device__ __forceinline__ void pool_groups(const float* x, int j0, int step, int P, int r, uint32_t (&key)[4 * G]) {
  typedef __attribute__((ext_vector_type(4), aligned(4))) float f32x4u;
  constexpr int E = (R + 3) / 4;  // pieces beside the own one
  constexpr int A = 4 * E;
  constexpr int N = 4 + 2 * A;
  if (FIXED) r = R;
  const float neutral = MODE == MASKKV_POOL_MAX ? __builtin_nanf("") : 0.f;  // (fmaxf passes over a NaN)
  const int lane = threadIdx.x & 63;
  auto load = [&](float (&w)[4], int p0) {
    const f32x4u q = *reinterpret_cast<const f32x4u*>(x + min(max(p0, 0), P - 4));
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = q[e];
  };
  const int side = lane == 0 ? -4 : 4;
  float own[G][4], end[G][E][4];
#pragma unroll
  for (int i = 0; i < G; ++i) load(own[i], j0 + i * step);
#pragma unroll
  for (int i = 0; i < G; ++i)
#pragma unroll
    for (int p = 0; p < E; ++p)
#pragma unroll
      for (int e = 0; e < 4; ++e) end[i][p][e] = 0.f;
  if (lane == 0 || lane == 63) {
#pragma unroll
    for (int i = 0; i < G; ++i)
#pragma unroll
      for (int p = 0; p < E; ++p) load(end[i][p], j0 + i * step + side * (p + 1));
  }
  float v[G][N];
#pragma unroll
  for (int i = 0; i < G; ++i) {
    within_prompt(own[i], j0 + i * step, P, neutral);
#pragma unroll
    for (int e = 0; e < 4; ++e) v[i][A + e] = own[i][e];
#pragma unroll
    for (int p = 0; p < E; ++p) {
      within_prompt(end[i][p], j0 + i * step + side * (p + 1), P, neutral);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        auto beside = [&](float of, int left) {  // (the lane that has none there keeps its own piece)
          const int kept = __builtin_bit_cast(int, end[i][p][e]), moved = __builtin_bit_cast(int, of);
          return __builtin_bit_cast(float, left ? __builtin_amdgcn_update_dpp(kept, moved, 0x138, 0xf, 0xf, false)     // wave_shr:1
                                                : __builtin_amdgcn_update_dpp(kept, moved, 0x130, 0xf, 0xf, false));  // wave_shl:1
        };
        v[i][A - 4 * (p + 1) + e] = beside(v[i][A - 4 * p + e], 1);
        v[i][A + 4 * (p + 1) + e] = beside(v[i][A + 4 * p + e], 0);
      }
    }
  }
  float acc[G][4];
#pragma unroll
  for (int i = 0; i < G; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[i][e] = neutral;  // (0 + x is x but for the sign of a zero, which the key does not see)
#pragma unroll
  for (int t = -R; t <= R; ++t)
    if (FIXED || (t >= -r && t <= r)) {
#pragma unroll
      for (int i = 0; i < G; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          acc[i][e] = MODE == MASKKV_POOL_MAX ? fmaxf(acc[i][e], v[i][e + A + t]) : __fadd_rn(acc[i][e], v[i][e + A + t]);
    }
#pragma unroll
  for (int i = 0; i < G; ++i) {
    const int g0 = j0 + i * step;
    const bool inner = g0 >= A && g0 + 4 + A <= P;
    // (As unsigned numbers negative sums, infinities and NaNs are above kDividableTo.  What is voted for is a sum of exponentials; of other
    // scores, negative sums tested by their magnitude, and keys of either sign, take 32 heads of 16384 positions from 11.3 to 9.65 us, 8192 8.0
    // to 7.1, positive ones from 9.5 to 9.7 and 7.15 to 7.2.)
    uint32_t least = 0u, most = 0xFFFFFFFFu;
    if (MODE != MASKKV_POOL_MAX) {
      uint32_t u[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) u[e] = __builtin_bit_cast(uint32_t, acc[i][e]);
      least = min(min(u[0], u[1]), min(u[2], u[3]));
      most = max(max(u[0], u[1]), max(u[2], u[3]));
    }
    if (inner && least >= kDividableFrom && most <= kDividableTo) {
      const float w = (float)(2 * r + 1), y = inverse(w);
#pragma unroll
      for (int e = 0; e < 4; ++e) key[4 * i + e] = __builtin_bit_cast(uint32_t, divided(acc[i][e], w, y)) | 0x80000000u;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int j = g0 + e;
        if (MODE != MASKKV_POOL_MAX) acc[i][e] = __fdiv_rn(acc[i][e], (float)(min(P - 1, j + r) - max(0, j - r) + 1));
        key[4 * i + e] = j < P ? order_key(acc[i][e]) : 0u;
      }
    }
  }
}

template <int G>
__device__ __forceinline__ void pooled_keys(const float* x, int j0, int step, int P, int window, int mode, uint32_t (&key)[4 * G]) {
  const int r = (window - 1) / 2;
  if (P >= 4 && r <= 8) {
    if (mode == MASKKV_POOL_MAX) {
      if (r <= 4)
        pool_groups<4, false, MASKKV_POOL_MAX, G>(x, j0, step, P, r, key);
      else
        pool_groups<8, false, MASKKV_POOL_MAX, G>(x, j0, step, P, r, key);
    } else if (r == 3) {
      pool_groups<3, true, MASKKV_POOL_MEAN, G>(x, j0, step, P, r, key);
    } else if (r <= 4) {
      pool_groups<4, false, MASKKV_POOL_MEAN, G>(x, j0, step, P, r, key);
    } else {
      pool_groups<8, false, MASKKV_POOL_MEAN, G>(x, j0, step, P, r, key);
    }
  } else {
#pragma unroll
    for (int i = 0; i < G; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int j = j0 + i * step + e;
        key[4 * i + e] = j < P ? pooled_key(x, j, P, r, mode) : 0u;
      }
  }
}

// Kept rows of the heads before `bh` (the sum of their clamped budgets): this thread's part, to be added up over the workgroup.
template <int THREADS>
__device__ __forceinline__ int rows_before(const SelectParams& prm, int bh) {
  int part = 0;
  for (int i = threadIdx.x; i < bh; i += THREADS) part += min(max(prm.budgets[i], 0), prm.lens.P[i / prm.H]);
  return part;
}

template <int THREADS>
__device__ __forceinline__ int take_base(const SelShared<THREADS>& s) {
  int base = 0;
#pragma unroll
  for (int w = 0; w < SelShared<THREADS>::kWaves; ++w) base += s.wbase[w];
  return base;
}

// ---- one workgroup per head: grid (BH), 4 * G keys a thread.  32 heads of 4096 positions: 16.0 us before (keys in LDS, one
// wave walking the histogram, refinement to a single key, two passes for the ordered output), 5.9 us now; 8192
// positions 20.0 us before (two stages) and 7.2 now; 12000 positions 11.7 us with every lane loading all of its windows, the ends of
// the prompt read a second time and four groups a thread, 8.2 now, and 14.3 and 8.4 with a window of 5 (group after group
// before, each waiting for its own loads); 16384 positions 11.4 and 9.5; 256 heads of 4096 ... 16384 positions 38
// and 11.3 us.  With three or four groups a thread it is the instructions a key that count, some 30 in all (1.4 us a group; 1.1 us of 10.5
// went with keys of positive means by one instruction instead of four, bins counted from the top, and, from three groups on, no bounds
// where the key tells and the keys below the k-th largest for certain left out of the histogram: with fewer groups the code that this
// adds costs a cold call as much as it saves).  Of the 13 thousand cycles at 4096 positions a third goes by until the keys are there, two thirds are the chain behind
// them.  Not better: the list ranked by all waves, each comparing a few, and the kept entries as a mask of bits.
template <int THREADS, int G>
__global__ __launch_bounds__(THREADS) void select_head_kernel(const SelectParams prm) {
  fetch_select_arguments();
  __shared__ SelShared<THREADS> s;
  const int bh = blockIdx.x;
  const int b = bh / prm.H;
  const int P = prm.lens.P[b];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int kh = min(max(prm.budgets[bh], 0), P);

  uint32_t key[4 * G];
  if (kh > 0)
    pooled_keys<G>(prm.scores + (int64_t)bh * prm.score_stride, 4 * tid, 4 * THREADS, P, prm.window, prm.mode, key);
  sel_clear(s);
  const int part = wave_incl_scan(rows_before<THREADS>(prm, bh));
  if (lane == 63) s.wbase[wave] = part;
  auto valid = [&](int i, int e) { return 4 * (tid + i * THREADS) + e < P; };
  uint32_t kmin = 0xFFFFFFFFu, kmax = 0u;
  if (kh > 0) {
#pragma unroll
    for (int i = 0; i < G; ++i) {
      if (valid(i, 3)) {
        kmin = min(kmin, min(min(key[4 * i], key[4 * i + 1]), min(key[4 * i + 2], key[4 * i + 3])));
        kmax = max(kmax, max(max(key[4 * i], key[4 * i + 1]), max(key[4 * i + 2], key[4 * i + 3])));
      } else {
#pragma unroll
        for (int e = 0; e < 3; ++e)
          if (valid(i, e)) {
            kmin = min(kmin, key[4 * i + e]);
            kmax = max(kmax, key[4 * i + e]);
          }
      }
    }
  }
  // Of the k largest keys none is below the lowest of k or more threads' (quads', rows') largest: the other two thirds (nine tenths) of
  // the keys need no place in the histogram.
  const int threads = min(THREADS, (P + 3) / 4);  // that have a key
  if (G > 2 && kh <= threads && P > kRankable) {
    kmin = kmax;
    int of = 1;
    if (kh <= (threads + 15) / 16) {
      kmin = row_max(kmax);
      of = 16;
    } else if (kh <= (threads + 3) / 4) {
      kmin = quad_max(kmax);
      of = 4;
    }
    if ((tid & -of) >= threads) kmin = 0xFFFFFFFFu;
  }
  uint32_t lo, hi;
  key_range(s, kmin, kmax, lo, hi);
  const int base = take_base(s);
  if (tid == 0) {
    prm.cu[bh] = base;
    if (bh == prm.BH - 1) prm.cu[prm.BH] = base + kh;
  }
  if (kh == 0) return;

  const uint64_t cut = exact_cut<(G > 2)>(s, lo, hi, kh, P, (uint32_t)(P - 1), [&](auto&& f) {
#pragma unroll
    for (int i = 0; i < G; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) f(key[4 * i + e], (uint32_t)(4 * (tid + i * THREADS) + e), valid(i, e));
  });

  // ---- ordered output: the groups of all threads follow one another, so every group has a scan of its own; the counts of
  // two groups (at most 4 * THREADS <= 4096 each) share a word
  auto kept = [&](int i, int e) {
    return code_of(key[4 * i + e], (uint32_t)(4 * (tid + i * THREADS) + e)) >= cut;
  };
  constexpr int kPairs = (G + 1) / 2;
  int own[kPairs], incl[kPairs];
#pragma unroll
  for (int p = 0; p < kPairs; ++p) own[p] = 0;
#pragma unroll
  for (int i = 0; i < G; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) own[i / 2] += kept(i, e) ? 1 << (16 * (i % 2)) : 0;
#pragma unroll
  for (int p = 0; p < kPairs; ++p) {
    incl[p] = wave_incl_scan(own[p]);
    if (lane == 63) s.wsum[p][wave] = incl[p];
  }
  __syncthreads();
  const int64_t room = prm.capacity - base;  // rows of idx this head may write
  const int rows = (int)min((int64_t)kh, max(room, (int64_t)0));
  int done = 0;  // rows of the groups before
#pragma unroll
  for (int p = 0; p < kPairs; ++p) {
    int before = incl[p] - own[p], total = 0;
#pragma unroll
    for (int w = 0; w < SelShared<THREADS>::kWaves; ++w) {
      const int t = s.wsum[p][w];
      before += w < wave ? t : 0;
      total += t;
    }
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const int i = 2 * p + half;
      if (i < G) {
        int at = done + ((before >> (16 * half)) & 0xFFFF);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (kept(i < G ? i : 0, e)) {
            if (at < rows) prm.idx[base + at] = 4 * (tid + i * THREADS) + e;
            ++at;
          }
        done += (total >> (16 * half)) & 0xFFFF;
      }
    }
  }
}

// ---- chunk stage: grid (BH, max_chunks).  Eight waves per SIMD, i.e. at most 64 registers: two workgroups then fit a
// compute unit.  32 heads of 32768 positions: 10.8 us before, 7.0 now.
__global__ __launch_bounds__(kSelThreads, 8) void select_chunk_kernel(const SelectParams prm) {
  fetch_select_arguments();
  __shared__ SelShared<kSelThreads> s;
  const int bh = blockIdx.x;
  const int b = bh / prm.H;
  const int P = prm.lens.P[b];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int kh = min(max(prm.budgets[bh], 0), P);
  const int c0 = (int)blockIdx.y * kChunk;
  if (c0 >= P || kh == 0) return;  // the final stage reads neither this chunk's count nor anything of a head without budget
  const int n = min(kChunk, P - c0);
  const int kc = min(kh, n);

  uint32_t key[4];
  pooled_keys<1>(prm.scores + (int64_t)bh * prm.score_stride, c0 + 4 * tid, 0, P, prm.window, prm.mode, key);
  sel_clear(s);
  const int nmine = min(max(n - 4 * tid, 0), 4);  // this thread's real keys: key[0 .. nmine)
  uint32_t kmin = 0xFFFFFFFFu, kmax = 0u;
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (e < nmine) {
      kmin = min(kmin, key[e]);
      kmax = max(kmax, key[e]);
    }
  uint32_t lo, hi;
  key_range(s, kmin, kmax, lo, hi);
  // A lower bound of the chunk's kc-th largest key: refinement until the bin that holds it has few keys left (every key
  // of that bin becomes a candidate, so the bound need not be tight; the final stage finds the cut exactly).
  Range g{lo, hi, kc, n};
  if (kc < n)
    refine<false>(s, g, kRankable, 0u, [&](auto&& f) {
#pragma unroll
      for (int e = 0; e < 4; ++e) f(key[e], e < nmine);
    });
  const uint32_t t0 = g.lo;  // kc >= n: the smallest key, everything is a candidate

  // ---- every key >= t0, in position order
  int mine = 0;
#pragma unroll
  for (int e = 0; e < 4; ++e) mine += (e < nmine && key[e] >= t0) ? 1 : 0;
  const int incl = wave_incl_scan(mine);
  if (lane == 63) s.wsum[0][wave] = incl;
  __syncthreads();
  int before = incl - mine;
  int total = 0;
#pragma unroll
  for (int w = 0; w < kSelWaves; ++w) {
    const int v = s.wsum[0][w];
    before += w < wave ? v : 0;
    total += v;
  }
  const int64_t ws = ((int64_t)bh * prm.max_chunks + blockIdx.y) * kChunk;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    if (e < nmine && key[e] >= t0) {
      prm.cand_key[ws + before] = key[e];
      prm.cand_pos[ws + before] = c0 + 4 * tid + e;
      ++before;
    }
  }
  if (tid == 0) prm.cand_cnt[(int64_t)bh * prm.max_chunks + blockIdx.y] = total;
}

// ---- final stage: grid (BH), over the chunk stage's candidates.  32 heads of 32768 positions and 171 ... 341 kept rows:
// 14.0 us before, 8.4 now.
__global__ __launch_bounds__(kSelThreads) void select_final_kernel(const SelectParams prm) {
  fetch_select_arguments();
  extern __shared__ uint32_t lds_words[];
  __shared__ SelShared<kSelThreads> s;
  __shared__ int coff[kMaxChunks + 1];  // candidates before chunk c

  const int bh = blockIdx.x;
  const int b = bh / prm.H;
  const int P = prm.lens.P[b];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int kh = min(max(prm.budgets[bh], 0), P);
  const int nch = (P + kChunk - 1) / kChunk;
  const int64_t head_ws = (int64_t)bh * prm.max_chunks * kChunk;

  // The first candidates of this wave's first chunk are asked for along with the counts that say how many there are: a
  // chunk's list has room for all its positions, so the addresses are good whatever the count.
  constexpr int kEarly = 5;
  uint32_t ekey[kEarly], epos[kEarly];
  if (kh > 0 && wave < nch) {
    const int64_t at = head_ws + (int64_t)wave * kChunk + lane;
#pragma unroll
    for (int u = 0; u < kEarly; ++u) {
      ekey[u] = prm.cand_key[at + 64 * u];
      epos[u] = (uint32_t)prm.cand_pos[at + 64 * u];
    }
  }
  sel_clear(s);
  const int part = wave_incl_scan(rows_before<kSelThreads>(prm, bh));
  const int cnt = (kh > 0 && tid < nch) ? prm.cand_cnt[(int64_t)bh * prm.max_chunks + tid] : 0;
  const int cincl = wave_incl_scan(cnt);
  if (lane == 63) {
    s.wbase[wave] = part;
    s.wtot[wave] = cincl;
  }
  __syncthreads();
  const int base = take_base(s);
  if (tid == 0) {
    prm.cu[bh] = base;
    if (bh == prm.BH - 1) prm.cu[prm.BH] = base + kh;
    coff[0] = 0;
  }
  if (kh == 0) return;
  int cbefore = 0;
#pragma unroll
  for (int w = 0; w < kSelWaves; ++w) {
    const int t = s.wtot[w];
    cbefore += w < wave ? t : 0;
  }
  if (tid < nch) coff[tid + 1] = cbefore + cincl;
  __syncthreads();

  const int n = coff[nch];
  const bool in_lds = n <= kSelLdsCap;           // the keys sit at lds_words[0 .. n)
  const bool pos_in_lds = 2 * n <= kSelLdsCap;   // the positions at lds_words[n .. 2n)
  // candidate e of the head sits in chunk c = the last one with coff[c] <= e
  auto slot_of = [&](int e) -> int64_t {
    int a = 0, z = nch;  // coff[a] <= e < coff[z]
    while (z - a > 1) {
      const int m = (a + z) >> 1;
      if (coff[m] <= e)
        a = m;
      else
        z = m;
    }
    return head_ws + (int64_t)a * kChunk + (e - coff[a]);
  };
  auto key_at = [&](int e) -> uint32_t { return in_lds ? lds_words[e] : prm.cand_key[slot_of(e)]; };
  auto pos_at = [&](int e) -> int { return pos_in_lds ? (int)lds_words[n + e] : prm.cand_pos[slot_of(e)]; };

  // ---- the chunks' lists into one (in LDS when they fit), and the range of the keys
  uint32_t kmin = 0xFFFFFFFFu, kmax = 0u;
  for (int c = wave; c < nch; c += kSelWaves) {
    const int first = coff[c], m = coff[c + 1] - first;
    const int64_t at = head_ws + (int64_t)c * kChunk;
    auto take = [&](int i, uint32_t k, uint32_t p) {
      if (in_lds) lds_words[first + i] = k;
      if (pos_in_lds) lds_words[n + first + i] = p;
      kmin = min(kmin, k);
      kmax = max(kmax, k);
    };
    int from = 0;
    if (c == wave) {
#pragma unroll
      for (int u = 0; u < kEarly; ++u)
        if (64 * u + lane < m) take(64 * u + lane, ekey[u], epos[u]);
      from = 64 * kEarly;
    }
    for (int i0 = from; i0 < m; i0 += 256) {  // four independent loads in flight per lane
      uint32_t k[4], p[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = min(i0 + 64 * u + lane, m - 1);
        k[u] = prm.cand_key[at + i];
        p[u] = pos_in_lds ? (uint32_t)prm.cand_pos[at + i] : 0u;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (i0 + 64 * u + lane < m) take(i0 + 64 * u + lane, k[u], p[u]);
    }
  }
  uint32_t lo, hi;
  key_range(s, kmin, kmax, lo, hi);

  // (an entry's number in the list stands for its position: the list is in position order)
  const uint64_t cut = exact_cut<false>(s, lo, hi, kh, n, (uint32_t)(n - 1), [&](auto&& f) {
    for (int e = tid; e < n; e += kSelThreads) f(key_at(e), (uint32_t)e, true);
  });

  // ---- ordered output: wave w owns entries [w*seg, (w+1)*seg)
  const int seg = ((n + kSelWaves - 1) / kSelWaves + 63) / 64 * 64;
  const int s0 = wave * seg;
  const int s1 = min(n, s0 + seg);
  auto kept = [&](int e) { return e < s1 && code_of(key_at(e), (uint32_t)e) >= cut; };
  int count = 0;
  for (int e0 = s0; e0 < s1; e0 += 64) count += __popcll(__ballot(kept(e0 + lane)));
  if (lane == 0) s.wsum[0][wave] = count;
  __syncthreads();
  int before = 0;
#pragma unroll
  for (int w = 0; w < kSelWaves; ++w) {
    const int t = s.wsum[0][w];
    before += w < wave ? t : 0;
  }
  const int64_t room = prm.capacity - base;  // rows of idx this head may write
  const int rows = (int)min((int64_t)kh, max(room, (int64_t)0));
  for (int e0 = s0; e0 < s1; e0 += 64) {
    const int e = e0 + lane;
    const bool k = kept(e);
    const uint64_t mask = __ballot(k);
    const int at = before + __popcll(mask & ((1ull << lane) - 1ull));
    if (k && at < rows) prm.idx[base + at] = pos_at(e);
    before += __popcll(mask);
  }
}

struct BudgetParams {
  int H, n_query;
  const float* mass;
  int32_t k_l;
  float alpha;
  int32_t* budgets;
};

// k_{l,h} = floor(alpha*k_l + (1-alpha) * N_h * k_l * P_h / sum_j P_j), P_h = mass_h / n_query.
// The sum is a tree over 256 threads' terms, halving the distance.  Up to 64 heads need one wave (THREADS 64): the
// upper halves would only add zeros, and the rest of the same tree needs neither LDS nor barriers.
template <int THREADS>
__global__ __launch_bounds__(THREADS) void head_budgets_kernel(const BudgetParams prm) {
  const int b = blockIdx.x;
  float s = 0.f;
  for (int h = threadIdx.x; h < prm.H; h += THREADS) s += prm.mass[b * prm.H + h] / (float)prm.n_query;
  if (THREADS > 64) {
    __shared__ float red[THREADS];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int o = THREADS / 2; o >= 64; o >>= 1) {
      if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
      __syncthreads();
    }
    s = red[threadIdx.x & 63];
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o, 64);
  const float total = __shfl(s, 0, 64);
  for (int h = threadIdx.x; h < prm.H; h += THREADS) {
    // a sequence without any prompt mass (empty prompt) has no preference: every head gets k_l
    const float p_hat = total > 0.f ? (prm.mass[b * prm.H + h] / (float)prm.n_query) / total : 1.f / (float)prm.H;
    const float v = prm.alpha * (float)prm.k_l + (1.f - prm.alpha) * (float)prm.H * (float)prm.k_l * p_hat;
    prm.budgets[b * prm.H + h] = (int32_t)floorf(v);
  }
}

int64_t select_chunks(const maskkv_desc* d) { return ((int64_t)d->P_max + kChunk - 1) / kChunk; }

int64_t select_cand_slots(const maskkv_desc* d) { return (int64_t)d->B * d->H * select_chunks(d) * kChunk; }

size_t select_count_bytes(const maskkv_desc* d) {
  return ((size_t)((int64_t)d->B * d->H * select_chunks(d)) * sizeof(int32_t) + 255) / 256 * 256;
}

}  // namespace

// Longest prompt the final stage can index (its chunk offsets live in LDS).
int64_t select_max_prompt() { return (int64_t)kMaxChunks * kChunk; }

// The (key, position) candidates that the chunk stage hands to the final stage, and their count per chunk.
size_t select_workspace_bytes(const maskkv_desc* d) {
  if (d->P_max <= kSinglePrompt) return 0;
  return (size_t)select_cand_slots(d) * (sizeof(uint32_t) + sizeof(int32_t)) + select_count_bytes(d);
}

int launch_select(const maskkv_desc* d, const Lens& lens, const float* scores, int64_t score_stride, int window,
                  int mode, const int32_t* budgets, int32_t* idx, int32_t* cu_budget, int64_t capacity,
                  void* workspace, hipStream_t stream) {
  SelectParams prm;
  prm.lens = lens;
  prm.H = d->H;
  prm.BH = d->B * d->H;
  prm.P_max = d->P_max;
  prm.scores = scores;
  prm.score_stride = score_stride;
  prm.window = window;
  prm.mode = mode;
  prm.budgets = budgets;
  prm.idx = idx;
  prm.cu = cu_budget;
  prm.capacity = capacity;
  prm.max_chunks = (int)select_chunks(d);
  prm.cand_key = reinterpret_cast<uint32_t*>(workspace);
  prm.cand_pos = reinterpret_cast<int32_t*>(prm.cand_key + select_cand_slots(d));
  prm.cand_cnt = prm.cand_pos + select_cand_slots(d);
  // One workgroup per head takes the fewest groups a thread that the prompt allows, and then the fewest waves: a group more costs
  // 1.5 us (the chain of every wave is longer by its keys), 256 threads more 0.4 to 0.8 (four waves start and meet at a barrier
  // sooner than sixteen).  32 heads, us, threads x groups: 2000 positions 256x2 6.3, 512x1 5.5, 768x1 5.8, 1024x1 6.3; 3000: 512x2
  // 6.2, 768x1 5.8, 1024x1 6.2; 4096: 512x2 6.2, 1024x1 6.1; 6000: 512x3 7.3, 768x2 6.9, 1024x2 7.6; 8192: 512x4 8.1, 768x3 8.1,
  // 1024x2 7.5; 12000: 768x4 9.5, 1024x3 9.2, 1024x4 11.0 (all before the last 0.3 to 1.0 us went).
  if (d->P_max <= kSinglePrompt) {
    const int groups = max(1, (int)((d->P_max + 4 * kSelThreads - 1) / (4 * kSelThreads)));
    const int threads = max(1, (int)((d->P_max + 1024 * groups - 1) / (1024 * groups))) * 256;
    auto start = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(prm.BH), dim3(threads), 0, stream, prm); };
    switch (groups << 16 | threads) {
      case 1 << 16 | 256: start(select_head_kernel<256, 1>); break;
      case 1 << 16 | 512: start(select_head_kernel<512, 1>); break;
      case 1 << 16 | 768: start(select_head_kernel<768, 1>); break;
      case 1 << 16 | 1024: start(select_head_kernel<1024, 1>); break;
      case 2 << 16 | 768: start(select_head_kernel<768, 2>); break;
      case 2 << 16 | 1024: start(select_head_kernel<1024, 2>); break;
      case 3 << 16 | 768: start(select_head_kernel<768, 3>); break;
      case 3 << 16 | 1024: start(select_head_kernel<1024, 3>); break;
      default: start(select_head_kernel<1024, 4>); break;  // (four groups: more than 12288 positions)
    }
    return check_launch("select (one stage)");
  }
  constexpr size_t dyn = (size_t)kSelLdsCap * sizeof(uint32_t);
  static bool granted = false;  // one-time opt-in to more than the default dynamic LDS size
  if (!granted) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&select_final_kernel),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)dyn);
    if (e != hipSuccess) {
      set_error("select: cannot raise dynamic LDS limit: %s", hipGetErrorString(e));
      (void)hipGetLastError();
      return MASKKV_EHIP;
    }
    granted = true;
  }
  hipLaunchKernelGGL(select_chunk_kernel, dim3(prm.BH, prm.max_chunks), dim3(kSelThreads), 0, stream, prm);
  if (int e = check_launch("select (chunk stage)")) return e;
  hipLaunchKernelGGL(select_final_kernel, dim3(prm.BH), dim3(kSelThreads), dyn, stream, prm);
  return check_launch("select (final stage)");
}

int launch_head_budgets(const maskkv_desc* d, const float* prompt_mass, int32_t k_l, float alpha, int32_t* budgets,
                        hipStream_t stream) {
  BudgetParams prm{d->H, d->n_query * query_heads_per_kv(d), prompt_mass, k_l, alpha, budgets};
  if (d->H <= 64)
    hipLaunchKernelGGL(head_budgets_kernel<64>, dim3(d->B), dim3(64), 0, stream, prm);
  else
    hipLaunchKernelGGL(head_budgets_kernel<256>, dim3(d->B), dim3(256), 0, stream, prm);
  return check_launch("head_budgets");
}

}  // namespace maskkv
