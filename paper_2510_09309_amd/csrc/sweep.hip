// Mask-Voting scores in one sweep over the prompt's keys (see score.hip for the two-pass form and the definitions).
//
// A column sum I_j = sum_i exp(s_ij) / L_i needs the normaliser L_i of every row before the first column can be summed, so
// score.hip forms the logits twice.  Here they are formed once: a workgroup forms the exponentials of a chunk of 128 keys x 256
// voting rows, keeps them in registers (64 per lane), publishes the chunk's row sums, forms the next chunk, and by then
// the row sums of all chunks of that unit have arrived and the kept chunk is turned into column sums.
//
//   start kernel  row references (the response span's log-sum-exp), the rows' sums over the response keys in units of them (1
//                 but for the rounding of the reference) as the initial values of the sums, the voting rows packed in
//                 MFMA fragment order, and a table of every workgroup's chunks.
//   sweep kernel  one workgroup of eight waves (32 rows each) per compute unit.  The chunks of a head are with as many workgroups
//                 at the same time (a round, see Packing); a workgroup takes its chunk through all groups of 256 voting rows of
//                 the head, with the keys in LDS, and adds the groups' column sums in registers.
//
// A step is a matrix phase (the logits of the chunk and their exponentials) and a vector phase (row sums published, the chunk of the
// step before completed).  Waves 4-7 run half a step behind waves 0-3, one of each on a SIMD, kept so by a barrier per phase:
// the vector phase is mostly latency, which the other wave's matrix phase fills.
//
// Per step a workgroup loads 64 KB of packed rows (from L2, into registers, each fragment as soon as the last MFMA that read
// the old one is issued) and per chunk 32 KB of keys (direct transfers into a ring of four chunks, three chunks ahead, and at the
// end of the vector phase: earlier they delay the answers that it waits for, in the matrix phase they stall it).  Row sums are added
// with 64-bit integer atomics, 4 copies of each sum; a step later every wave reads the sums of its own rows.  Nothing
// waits for a sum that is not needed yet, and every wait is bounded: if the workgroups turn out not to be all resident, or a
// row's sum leaves the range of the integers, a two-pass fallback at the end of the same kernel does the work.
//
// What bounds it: a step of 5800 to 7100 cycles, 2048 of them MFMAs.  A wave issues an instruction every 4 to 5 cycles, a matrix phase
// has 1800 cycles of them, a vector phase 1300 to 1800, and the two waves of a SIMD share the vector pipe, where v_exp_f32
// takes 8 cycles and an MFMA about as many.  In a loop of nothing but long calls the board is at its 1400 W and the clock 10 % below that
// of short calls (2.1 against 2.3 GHz); as part of a layer the sweep is below that.  us a call, with both groups of waves in the same
// phase, chunks dealt out end to end and keys transferred for every group of rows before: 32 heads x 128 with 256 rows, 4k keys 28.7
// -> 27.1, 8k 39 -> 36.6, 32k 120 -> 114; 4 heads with 1792 rows over 30k keys 93.5 -> 87.4; the ragged batch of perf/cases.py 518 ->
// 466 (8 more with 64-bit addresses formed for every access, 6 more with the start kernel's loads in turn).  (Without transfers of keys, with
// wrong results, the ragged batch took 420 instead of 505, without loads of rows 455, without the exchange 465.)  Slower: raised
// wave priority in the vector phase or for waves 4-7; a first sum per XCD that the last of its workgroups adds to the whole
// (two latencies instead of one); 2 or 8 copies of the sums.
#include <type_traits>

#include "kernels.hpp"
#include "lds.hpp"
namespace maskkv {

namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int kRows = 256;                 // voting rows per unit at most; a unit is one (sequence, head, group of voting rows)
constexpr int kWaves = 8;                  // each owns 32 rows
constexpr int kThreads = 64 * kWaves;
constexpr int kNB = 4;                     // 32-key blocks per chunk
constexpr int kKeys = 32 * kNB;
constexpr int kAhead = 3;                  // slots between the LDS read of a fragment and its use
constexpr int kLag = 2;                    // slots between the last MFMA of a block and its first exponential
constexpr int kCopies = 4;                 // of every row's `low` sum: workgroups spread their additions over them

// Row sums are exchanged as integers, so that their total does not depend on the order of arrival: 10 bits count the chunks
// that have been added, 54 bits hold the sum in units of 2^-28 of the response span's own sum (`low`) or, for a chunk
// whose sum is 2^16 of it or more, in units of 2^-7 (`high`), which are the last place of such a sum in fp32 or smaller.
constexpr int kCountShift = 54;
constexpr uint64_t kSumMask = (1ull << kCountShift) - 1;
constexpr float kLowScale = 268435456.f;   // 2^28
constexpr float kLowLimit = 65536.f;       // 2^16
constexpr float kHighScale = 128.f;        // 2^7
constexpr float kHighLimit = 549755813888.f;  // 2^39 (kMaxGroups chunks below either limit stay below 2^54 units)
constexpr uint64_t kTaskWait = 100000000;  // 1 s of the 100 MHz clock: a task of the fallback for tasks that are being done

// A row's mass is its prompt sum over its whole sum.  The former comes out of the exchange with an error of about 1e-8 (256
// chunks rounded to units of 2^-28) and of the rounding of the row's reference, 1e-7 to 1e-6 of the response span's sum: below fp32's
// own error only as long as the prompt's share is not small.  Where more of a wave's 32 rows have a whole sum below kSmallSum than
// above, the mass of these rows is taken from the column sums instead, which are as accurate as fp32 however small they are:
// that wave of every chunk's workgroup (all see the same row sums, so they agree) leaves the sum of its part of the column
// sums, and the workgroup of the unit's leading chunk adds these up in a fixed order after its walk.  (Within what two runs
// differ by, a call without such waves takes the time it took when every mass came from the row sums.)
constexpr float kSmallSum = 2.f;
constexpr float kNoRow = 0.5f;             // whole sum of a row that does not exist (its mass is then cut off at 0; a row that does has 1)
constexpr uint32_t kNoPart = 0xFFFFFFFFu;  // not there (a part has its sign bit clear)

constexpr int kMaxUnits = 4096;            // of a launch, see sweep_plan
constexpr int kMaxGroups = 256;            // workgroups of a sweep, and chunks of a unit, at most (one per compute unit)

// What a unit has in the workspace, one behind the other, so that a base and 32 bits address all of it:
//   row sums  [kCopies][256] `low`, [256] `high` (64 bits each)
//   [8 waves][2][32] floats: the rows' references, minus the response span's log-sum-exp in units of the raw logits; and the sums
//   of the response span in units of these references, 1 but for their rounding
//   [8 waves] 32 rows in MFMA fragment order
constexpr uint32_t kHighAt = kCopies * kRows * 8, kRefsAt = kHighAt + kRows * 8, kRowsAt = kRefsAt + kWaves * 256;
template <int D>
constexpr uint32_t kUnitBytes = kRowsAt + kRows * D * 2;
static_assert((uint64_t)kMaxUnits * kUnitBytes<128> <= 0xFFFFFFFFu, "a unit's place is held in 32 bits (Task::at)");

struct Control {
  int run;      // this call's workgroups may be placed as a sweep's
  int redo;     // the sweep could not do the work: the fallback at the end of the kernel does
  int ticket;   // next task of the fallback
};

constexpr int kSpans = 8;                  // pieces of a unit's keys in the fallback's first pass, at most
constexpr int kSpanChunks = 8;             // chunks of a piece in its second pass where a head has several groups of rows, at most

// A chunk of a head's keys.
struct __attribute__((aligned(16))) Chunk {
  int bh;
  uint32_t shape;     // its number, 8 bits; the head's number of chunks less one, 8 bits; its number of keys, or 0: none (HALVES)
  const char* keys;
  float* out;         // its scores
  int64_t pad;
};

struct SweepParams {
  View Q, K;
  Lens lens;
  int B, H, n_resp;
  int n_query;      // voting rows per key/value head: q_per_kv query heads of n_qh mask queries each
  int n_qh, q_per_kv;
  int subsets;      // of a head's groups of voting rows; each counts as a head of its own, with the same keys
  int nqg;          // groups of a subset
  int rows;         // voting rows per unit, a multiple of 32 (the last unit of a head may have fewer)
  SweepPlan plan;
  struct Chunk* table;  // [groups][rounds] what a workgroup's chunks are, in turn
  int* counts;          // [groups] how many they are
  int tables;           // workgroups of the start kernel that fill the table, a wave a head
  int rounds;
  int patience;     // how long a workgroup waits for the others' row sums, in ticks of the 100 MHz clock
  int spans;        // pieces of a unit's keys in the fallback's first pass
  int spans2;       // pieces of a head's keys in its second pass
  float c;          // scale * log2(e)
  char* units;      // [units][unit_bytes], see kHighAt
  Control* ctl;
  int* spans_done;  // [units] spans of the unit whose statistics are there (fallback)
  uint32_t* parts;  // [units][8 waves][n_parts] bits of a chunk's part of the mass of 32 rows, or kNoPart
  int n_parts;      // chunks of the longest prompt
  int* late;        // [B*H*subsets] 1 + the next head of a workgroup's list for late_masses, or 0
  float2* stats;    // [units][spans][256] (reference, sum) of a span of chunks (fallback)
  float* out;       // [B*H*subsets][out_stride]
  int64_t out_stride;
  float* mass;      // [B*H*subsets] or null
  __device__ int heads() const { return H * subsets; }  // of a sequence, subsets counted as heads
};

__device__ __forceinline__ void fetch_sweep_arguments() {
  typedef SweepParams A;
  fetch_arguments({MASKKV_VIEW_ARGUMENTS(A, Q), MASKKV_VIEW_ARGUMENTS(A, K), MASKKV_ARGUMENT(A, lens), MASKKV_ARGUMENT(A, B), MASKKV_ARGUMENT(A, n_qh),
                   MASKKV_ARGUMENT(A, plan.places), MASKKV_ARGUMENT(A, plan.heads), MASKKV_ARGUMENT(A, table), MASKKV_ARGUMENT(A, patience),
                   MASKKV_ARGUMENT(A, units), MASKKV_ARGUMENT(A, parts), MASKKV_ARGUMENT(A, out)});
}

// The workgroups of a sweep wait for each other, so all of them have to be resident, and two sweeps may not be placed on a device at
// the same time.  The lock holds how many workgroups all sweeps together have been or are to be placed (32 bits, wrapping),
// and when it was last changed (32 bits, in kTick); what has been placed counts itself in 16 places, since 256 additions to one
// word at the beginning of a sweep hold it up by 10 us.  A call adds its workgroups in its start kernel.  At no difference
// between the two the next sweep may line up behind this one; while there is one its start kernel waits, which
// keeps that compute unit from the others: it goes on when no more than kWaiters are to come.  These have waited for a
// place since before this call's sweep is launched, so they come first.  After kStartWait the call takes the fallback.
// If a sweep kernel never runs, because its launch failed or a graph was given up, its workgroups are forgotten kStale
// later; a call that is merely slow then loses nothing but time, since all waits are bounded.
// The lock is a variable of this library: other processes on the device, or a second copy of the library, have their own, and other
// kernels may hold compute units as well (a workgroup needs 145 KB of LDS and, at head_dim 128, all registers).  Workgroups that are
// kept apart that way give up after `patience`, and those that run do the work in the fallback.
// us a call on two streams at once (one stream; the fallback for whoever finds the lock taken; the two passes): 4k keys 24, 28, 31, 30;
// 8k 38, 40, 40, 58; 32k 119, 121, 168, 162; 8 sequences x 8k with 512 rows 445, 454, 605, 648.  Six threads with a stream each: 4k 24
// (30 with the two passes), 32k 200 (146: with several waiting at once most calls take the fallback; 240 with waits of 500 us).
__device__ unsigned long long sweep_lock;
constexpr int kPlaces = 16;
constexpr int kPlaceWords = 32;            // (a line each)
__device__ unsigned sweep_placed[kPlaces * kPlaceWords];
constexpr int kWaiters = 8;
constexpr int kTick = 20;                  // 2^20 ticks of the 100 MHz clock: 10 ms
constexpr uint32_t kStale = 100;           // 1 s
// 100 us.  Longer gains nothing (25 us are enough for two streams, and a start kernel that waits behind the same hardware queue as the
// sweep it waits for, or that keeps a place from it beside other waiting ones, waits in vain), 10 us is too short.
constexpr uint64_t kStartWait = 10000;

__device__ __forceinline__ uint32_t placed() {  // by all sweeps (to be called by a whole wave)
  const int lane = threadIdx.x & 63;
  uint32_t v = lane < kPlaces ? __hip_atomic_load(&sweep_placed[lane * kPlaceWords], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Adds a call's workgroups if no more than most_left are to come (to be called by a whole wave; the same in every lane).
__device__ __forceinline__ bool take_lock(int groups, int most_left) {
  unsigned long long seen = __hip_atomic_load(&sweep_lock, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const uint32_t there = placed();  // (it only grows: at worst too many seem to be left)
  const uint32_t now = (uint32_t)(wall_clock64() >> kTick);
  const bool stale = now - (uint32_t)(seen >> 32) - 1 < 0x7FFFFFFFu && now - (uint32_t)(seen >> 32) > kStale;
  const int left = (int)((uint32_t)seen - there);
  if (left > most_left && !stale) return false;
  const uint32_t all = (left > 0 && !stale ? (uint32_t)seen : there) + (uint32_t)groups;
  unsigned long long was = 0;
  if ((threadIdx.x & 63) == 0) was = atomicCAS(&sweep_lock, seen, ((unsigned long long)now << 32) | all);
  return __all((threadIdx.x & 63) != 0 || was == seen);
}

__device__ __forceinline__ int ceil_div(int a, int b) { return (a + b - 1) / b; }

template <int D>
struct Cfg {
  static constexpr int kRowB = D * 2;
  static constexpr int kRing = 4;                   // chunks of keys in LDS
  static constexpr int kSteps = kRowB / 32;
  static constexpr int kPPR = kRowB / 16;           // 16-byte pieces per row
  static constexpr int kRPI = 1024 / kRowB;         // rows moved by one wave instruction
  static constexpr int kMoves = kKeys / kWaves / kRPI;  // transfers per wave and chunk
  static constexpr int kKBytes = kKeys * kRowB;
  static constexpr int kQBytes = 32 * kRowB;        // per wave
  static constexpr int kOffStart = kRing * kKBytes; // behind the ring of chunks: [2][kWaves][64] floats (fallback: [kSpanChunks][kKeys])
  static_assert(kSpanChunks * kKeys == 2 * kWaves * 64, "a piece's column sums take the references' place");
  static constexpr int kOffCs = kOffStart + 2 * kWaves * 256;  // [2][kWaves][kKeys] floats
  static constexpr int kOffW = kOffCs + 2 * kWaves * kKeys * 4;  // [kWaves][32] floats
  static constexpr int kOffInf = kOffW + kWaves * 128;         // 32 floats: -inf
  static constexpr int kOffMass = kOffInf + 128;               // [2][kWaves] floats
  static constexpr int kOffBad = kOffMass + 2 * kWaves * 4;    // one int: the scores of this workgroup are void
  static constexpr int kOffLate = kOffBad + 4;                 // two ints: 1 + the first head that late_masses has to do, or 0
  static constexpr int kOffRedo = kOffBad + 12;                // one int: another workgroup's are
  static constexpr int kLds = kOffBad + 64;
  // Rows are stored without padding (a direct transfer writes 1 KiB of consecutive LDS); piece p of row r sits in
  // slot p ^ swz(r), which spreads the fragment reads of 16 consecutive rows over all banks.
  __device__ static int swz(int row) { return D == 128 ? row & 15 : (row >> 1) & 7; }
};

__device__ __forceinline__ uint64_t peek(Base b, uint32_t off) {
  return __hip_atomic_load(at<uint64_t>(b, off), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ bool mostly_small(float L) {  // the same in every lane of a wave
  const uint64_t small = __ballot(fabsf(L - 0.5f * (0.75f + kSmallSum)) < 0.5f * (kSmallSum - 0.75f));  // (but not kNoRow)
  return __popcll(small) > __popcll(__ballot(L >= kSmallSum));
}
__device__ __forceinline__ float row_mass(float L, float inv) { return fmaxf(L - 1.f, 0.f) * inv; }
// the reciprocal of a row's sum
__device__ __forceinline__ float reciprocal(float L) {
  const float w = __builtin_amdgcn_rcpf(L);
  return fmaf(fmaf(-L, w, 1.f), w, w);
}
__device__ __forceinline__ float whole(uint64_t v) {  // an exchanged sum without the count
  return fmaf((float)((uint32_t)(v >> 32) & ((1u << (kCountShift - 32)) - 1)), 4294967296.f, (float)(uint32_t)v);
}

template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, false));
}

// The sum over a wave, in every lane, without the LDS.
__device__ __forceinline__ float wave_sum(float v) {
  v += dpp<0xB1>(v);   // neighbours
  v += dpp<0x4E>(v);   // pairs
  v += dpp<0x141>(v);  // half rows, mirrored
  v += dpp<0x140>(v);  // rows of 16, mirrored
  const auto a = __builtin_amdgcn_permlane16_swap(as_u32(v), as_u32(v), false, false);
  const unsigned a0 = a[0], a1 = a[1];
  v = as_f32(a0) + as_f32(a1);
  const auto b = __builtin_amdgcn_permlane32_swap(as_u32(v), as_u32(v), false, false);
  const unsigned b0 = b[0], b1 = b[1];
  return as_f32(b0) + as_f32(b1);
}

// The sum of the waves' masses, by halves: in turn, the last additions would each round as much as the whole does (two sequences of 14k and
// 24k keys: errors against 64 bits of 4.3e-8, the two passes 3.2e-8).
template <int N>
__device__ __forceinline__ float sum_of_waves(uint32_t lds) {
  float v[N];
#pragma unroll
  for (int w = 0; w < N; ++w) v[w] = *in_lds<const float>(lds, w * 4);
#pragma unroll
  for (int n = N / 2; n > 0; n /= 2)
#pragma unroll
    for (int w = 0; w < n; ++w) v[w] += v[w + n];
  return v[0];
}

// The plan's runs in the lanes of a wave: what a loop over them reads is then a register of the wave's instead of a scalar load that it
// waits for (all of them once; a round of the loop costs the waits 0.3 us).
struct Runs {
  uint32_t places[kMaxRuns / 64], heads[kMaxRuns / 64], repeats[kMaxRuns / 64];
  int n;
  bool halves;
  __device__ __forceinline__ explicit Runs(const SweepPlan& plan) : n(plan.runs), halves(plan.halves()) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int k = 0; k < kMaxRuns / 64; ++k)
      if (k == 0 || n > 64 * k) {
        places[k] = plan.places[64 * k + lane];
        heads[k] = plan.heads[64 * k + lane];
        repeats[k] = plan.repeats[64 * k + lane];
        asm volatile("" : "+v"(places[k]), "+v"(heads[k]), "+v"(repeats[k]));  // (here, where all lanes are: others read them later)
      }
  }
  static __device__ __forceinline__ uint32_t of(const uint32_t (&v)[kMaxRuns / 64], int i) {
    uint32_t x = (uint32_t)__builtin_amdgcn_readlane((int)v[0], i & 63);
#pragma unroll
    for (int k = 1; k < kMaxRuns / 64; ++k)
      if (i >= 64 * k) x = (uint32_t)__builtin_amdgcn_readlane((int)v[k], i & 63);
    return x;
  }
  // The run that serves a head of a sequence, or n.
  __device__ __forceinline__ int serving(int b, int h) const {
    const int lane = threadIdx.x & 63;
    int i = n;
#pragma unroll
    for (int k = kMaxRuns / 64 - 1; k >= 0; --k)
      if (k == 0 || n > 64 * k) {
        const int from = heads[k] & 0xFFFF, side = heads[k] >> 16, times = repeats[k] & 0xFFFF;
        const uint64_t they =
            __builtin_amdgcn_ballot_w64(64 * k + lane < n && (int)(repeats[k] >> 16) == b && h >= from && h < from + side * times);
        if (they) i = 64 * k + __builtin_ctzll(they);
      }
    return i;
  }
  // Calls each(w has a chunk in it, its repetitions) for the rounds that end before run i.
  template <typename Each>
  __device__ __forceinline__ void rounds(int i, int w, Each&& each) const {
    bool has = false;
    uint32_t times = 0;
    for (int j = 0; j < i; ++j) {
      const uint32_t place = of(places, j);
      const int at = place & 0xFFFF;
      if (at == 0 || j == 0) {
        if (j > 0) each(has, (int)times);
        has = false;
        times = of(repeats, j) & 0xFFFF;
      }
      has = has || (w >= at && w < at + (int)(place >> 16));
    }
    // (the round that run i belongs to may have begun before it)
    if (i > 0 && (i == n || (of(places, i) & 0xFFFF) == 0)) each(has, (int)times);
  }
};

// Takes the lock, or waits for it (2 us), and counts every workgroup's chunks: for a workgroup of its own, the first, so that this is
// over when the others are.
__device__ __forceinline__ void start_lock(const SweepParams& prm) {
  const Runs runs(prm.plan);
  const int w = threadIdx.x;
  int n = 0;
  runs.rounds(runs.n, w, [&](bool has, int times) {
    if (!has && runs.halves && w < prm.plan.groups) {
      Chunk c;
      c.bh = 0;
      c.shape = 0;
      c.keys = prm.K.row(0, 0, 0);
      c.out = prm.out;
      for (int t = n; t < n + times; ++t) prm.table[(int64_t)w * prm.rounds + t] = c;
    }
    n += has || runs.halves ? times : 0;
  });
  if (w < prm.plan.groups) prm.counts[w] = n;
  if (threadIdx.x >= 64) return;
  bool run = take_lock(prm.plan.grid, 0);
  const uint64_t t0 = wall_clock64();
  while (!run && wall_clock64() - t0 < kStartWait) {
    __builtin_amdgcn_s_sleep(32);
    run = take_lock(prm.plan.grid, kWaiters);
  }
  if (threadIdx.x == 0) {
    prm.ctl->run = run;
    prm.ctl->redo = !run;
    prm.ctl->ticket = 0;
  }
}

// The table's entries of a head (to be called by a whole wave).
__device__ __forceinline__ void start_table(const SweepParams& prm, int b, int vh) {
  const Runs runs(prm.plan);
  const int lane = threadIdx.x & 63;
  const int P = prm.lens.P[b], nc = (P + kKeys - 1) / kKeys;
  const int i = runs.serving(b, vh);
  if (i == runs.n) return;  // (no prompt)
  const uint32_t heads = Runs::of(runs.heads, i);
  const int nth = vh - (int)(heads & 0xFFFF), side = heads >> 16;
  const int w0 = (int)(Runs::of(runs.places, i) & 0xFFFF) + nth % side * nc;
  for (int c0 = 0; c0 < nc; c0 += 64) {
    const int ci = c0 + lane, w = w0 + ci;
    int t = nth / side;
    runs.rounds(i, w, [&](bool has, int times) { t += has || runs.halves ? times : 0; });
    Chunk c;
    c.bh = b * prm.heads() + vh;
    c.shape = (uint32_t)ci | (uint32_t)(nc - 1) << 8 | (uint32_t)min(P - ci * kKeys, kKeys) << 16;
    c.keys = prm.K.row(b, vh / prm.subsets, (int64_t)ci * kKeys);
    c.out = prm.out + (int64_t)c.bh * prm.out_stride + ci * kKeys;
    if (ci < nc) prm.table[(int64_t)w * prm.rounds + t] = c;
  }
}

// ---- response span: row references, zeroed sums, and the voting rows in the order in which the sweep reads them.
// A workgroup serves BLOCKS blocks of 32 rows of a unit; 8 / BLOCKS waves share a block's keys, which come through LDS 128
// at a time.  Eight blocks where there are units enough to fill the chip (each key is then read once per unit), otherwise two.
//
// What bounds it: with few units the latency of its loads (issued at once: rows and two tiles of keys; 5.9 to 6.7 us with the rest of the
// chain: launch, loads, logarithms, stores), with many the memory (96 MB in the ragged batch of perf/cases.py, 20 of 35 us) and
// the exponentials (12 us), which all workgroups come to at the same time.  us there, 40.6 -> 35: the sweep's table written by
// workgroups of their own instead of by a wave that the others wait for, tiles asked for before the rows' arrival instead of
// after it, the packed rows stored after the last wait, masks only where the span ends.  8 sequences of 32 heads with 69 rows: 51 -> 48
// for the whole call, 6 of 28 with 116 rows 36.4 -> 33.0.  Not better: units dealt to the XCDs by head, four blocks a workgroup (39).
template <int D, int BLOCKS>
__global__ __launch_bounds__(kThreads) void sweep_start_kernel(const SweepParams prm) {
  using C = Cfg<D>;
  fetch_sweep_arguments();
  constexpr int S = C::kSteps, SPLIT = kWaves / BLOCKS;
  constexpr bool kShared = BLOCKS < 8;
  const int lane = threadIdx.x & 63, r = lane & 31, g = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if ((int)blockIdx.x <= prm.tables) {
    if (blockIdx.x == 0) {
      start_lock(prm);
    } else {
      const int head = ((int)blockIdx.x - 1) * kWaves + wave;
      if (head < prm.B * prm.heads()) start_table(prm, head / prm.heads(), head % prm.heads());
    }
    return;
  }
  extern __shared__ __attribute__((aligned(1024))) char lds[];  // two tiles of 128 keys, and with kShared the rows
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;
  float2(&part)[kWaves][32] = *reinterpret_cast<float2(*)[kWaves][32]>(lds + 2 * C::kKBytes);  // (in the rows' place: two workgroups fit a compute unit)
  const int block = (int)blockIdx.x - 1 - prm.tables;
  const int unit = block / SPLIT;
  // (a division is a chain of some twenty instructions before the first load)
  const int bh = prm.nqg == 1 ? unit : unit / prm.nqg;
  const int b = prm.B == 1 ? 0 : bh / prm.heads(), vh = bh - b * prm.heads();
  const int h = prm.subsets == 1 ? vh : vh / prm.subsets;
  const int qg = (vh - h * prm.subsets) * prm.nqg + unit - bh * prm.nqg;
  const int P = prm.lens.P[b];
  const char* keys = prm.K.row(b, h, P);
  auto dma = [&](int t) {
    // (a tile's rows are up to 127 x 16 MiB apart and fit 32 bits, those of the whole span do not)
    const char* base = keys + (int64_t)(t * kKeys) * prm.K.stride_t;
    const int last = prm.n_resp - 1 - t * kKeys;
#pragma unroll
    for (int j = 0; j < C::kMoves; ++j) {
      const int row = wave * (kKeys / kWaves) + j * C::kRPI + lane / C::kPPR;
      const int piece = (lane % C::kPPR) ^ C::swz(row);
      dma16(base, (uint32_t)min(row, last) * (uint32_t)prm.K.stride_t + piece * 16,
            lds0 + (t & 1) * C::kKBytes + (wave * (kKeys / kWaves) + j * C::kRPI) * C::kRowB);
    }
  };
  const int tiles = ceil_div(prm.n_resp, kKeys);
  const int rb = block % SPLIT * BLOCKS + wave / SPLIT;  // block of 32 rows
  const int part_of = wave % SPLIT;
  const int q0 = qg * prm.rows + rb * 32;
  u32x4 qf[S];
  const uint32_t rows = lds0 + 2 * C::kKBytes + wave / SPLIT * C::kQBytes;  // (behind the tiles)
  // Two blocks: a block's waves move its rows as whole rows, each row once.  (Each wave loading the fragments of all its rows, a row a
  // lane, keeps the texture path busy for four times as long, and that four times over: first data after 3.4 us of 5.2 instead of 2.2
  // of 4.2; us a layer 4k keys 45.6 -> 44.4, 8k 57.8 -> 56.8, two sequences of 3k and 5k at head_dim 64 41.3 -> 40.3, 8 heads x 410 x 4 rows, 4.7k
  // keys, scoring alone 45.3 -> 44.3.  Eight blocks have too little LDS for it, or one more wait: the ragged batch takes the same.)
  if (kShared) {
#pragma unroll
    for (int j = 0; j < C::kQBytes / 1024 / SPLIT; ++j) {
      const int row = (part_of * (C::kQBytes / 1024 / SPLIT) + j) * C::kRPI + lane / C::kPPR;
      const char* from = prm.Q.group_row(b, h, prm.q_per_kv, prm.n_qh, min(q0 + row, prm.n_query - 1));
      dma16_from(from + ((lane % C::kPPR ^ C::swz(row)) << 4), rows + (part_of * (C::kQBytes / 1024 / SPLIT) + j) * 1024);
    }
  } else {
    const char* qrow = prm.Q.group_row(b, h, prm.q_per_kv, prm.n_qh, min(q0 + r, prm.n_query - 1)) + g * 16;
#pragma unroll
    for (int s = 0; s < S; ++s) asm volatile("global_load_dwordx4 %0, %1, off offset:%2" : "=v"(qf[s]) : "v"(qrow), "i"(s * 32));
  }
  dma(0);
  if (tiles > 1) dma(1);

  char* area = prm.units + (int64_t)unit * kUnitBytes<D>;
  uint64_t* sums = reinterpret_cast<uint64_t*>(area) + rb * 32;
  float m = kNegBig, l = 0.f;
  for (int t = 0; t < tiles; ++t) {
    if (t + 1 < tiles)
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"i"(C::kMoves) : "memory");
    else
      asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (kShared && t == 0)
#pragma unroll
      for (int s = 0; s < S; ++s) qf[s] = *in_lds<const u32x4>(rows + r * C::kRowB + (((2 * s + g) ^ C::swz(r)) << 4));
#pragma unroll
    for (int s = 0; s < S; ++s) asm volatile("" : "+v"(qf[s]));
    if (t + 1 == tiles && part_of == 0) {  // (stores before the last wait would be waited for)
      if (lane < 32) {
#pragma unroll
        for (int i = 1; i <= kCopies; ++i) sums[i * kRows + lane] = 0;  // (the last one is `high`)
      }
      for (int i = lane; i < ceil_div(P, kKeys); i += 64) prm.parts[((int64_t)unit * kWaves + rb) * prm.n_parts + i] = kNoPart;
      u32x4* pack = reinterpret_cast<u32x4*>(area + kRowsAt + rb * C::kQBytes) + lane;
#pragma unroll
      for (int s = 0; s < S; ++s) pack[s * 64] = qf[s];
      if (rb == 0 && lane == 0) {
        prm.spans_done[unit] = 0;
        if (P == 0 && prm.mass) prm.mass[bh] = 0.f;
      }
    }
    for (int kb = part_of; kb < kNB; kb += SPLIT) {
      const int k0 = t * kKeys + kb * 32;
      if (k0 >= prm.n_resp) break;
      f32x16 a{};
#pragma unroll
      for (int s = 0; s < S; ++s) {
        const u32x4 kf = *in_lds<const u32x4>(lds0 + (t & 1) * C::kKBytes + (kb * 32 + r) * C::kRowB + (((2 * s + g) ^ C::swz(r)) << 4));
        mfma_step<bf16_t>(kf, qf[s], a);
      }
      if (k0 + 32 > prm.n_resp)
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (k0 + 8 * (i / 4) + 4 * g + (i % 4) >= prm.n_resp) a[i] = -INFINITY;
      float top = a[0];
#pragma unroll
      for (int i = 1; i < 16; ++i) top = fmaxf(top, a[i]);
      const float m_new = fmaxf(m, top * prm.c);
      float s0 = 0.f, s1 = 0.f;
#pragma unroll
      for (int i = 0; i < 16; i += 2) {
        s0 += fast_exp2(fmaf(a[i], prm.c, -m_new));
        s1 += fast_exp2(fmaf(a[i + 1], prm.c, -m_new));
      }
      l = l * fast_exp2(m - m_new) + (s0 + s1);
      m = m_new;
    }
    if (t + 2 < tiles) {
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
      dma(t + 2);
    }
  }
  {
    const float mo = xor32(m), lo = xor32(l);
    const float mm = fmaxf(m, mo);
    l = l * fast_exp2(m - mm) + lo * fast_exp2(mo - mm);
    m = mm;
  }
  if (SPLIT > 1) {
    if (tiles == 1) __syncthreads();  // (every wave has its rows)
    if (g == 0) part[wave][r] = make_float2(m, l);
    __syncthreads();
  }
  if (part_of == 0 && lane < 32) {
    if (SPLIT > 1) {
      float M = kNegBig, L = 0.f;
#pragma unroll
      for (int w = 0; w < SPLIT; ++w) M = fmaxf(M, part[wave + w][lane].x);
#pragma unroll
      for (int w = 0; w < SPLIT; ++w) L += part[wave + w][lane].y * fast_exp2(part[wave + w][lane].x - M);
      m = M;
      l = L;
    }
    // The logarithm and its sum with m carry what they lost along; what the rounding of the reference itself loses is in `own`.
    const float lg = __log2f(l), near1 = l * fast_exp2(-lg);
    const float sum = m + lg, back = sum - m;
    const float lost = (m - (sum - back)) + (lg - back);
    const bool live = rb * 32 < prm.rows && q0 + lane < prm.n_query;
    const float ref = -(sum + (lost + (near1 - 1.f) * kLog2e)) / prm.c;
    const float own = live ? near1 * fast_exp2(fmaf(ref, prm.c, sum) + lost) : kNoRow;
    float* refs = reinterpret_cast<float*>(area + kRefsAt) + rb * 64 + lane;
    refs[0] = live ? ref : -INFINITY;
    refs[32] = own;
    sums[lane] = (uint64_t)rintf(own * kLowScale);
  }
}

// ---- fallback: the scores in two passes, as tasks that workgroups take by ticket, whatever their number.  A task is a
// span of a unit's chunks; first come all tasks that form row statistics, then all that form column sums.  The latter wait
// for the former of their unit, which have smaller tickets and therefore are with workgroups that are running.
//
// A call comes here if a row's sum is out of range, if the device's sweep stays taken, or if another program's kernels keep its
// workgroups apart, so it is no mere safety net: keys come by direct transfers two chunks ahead, with one barrier a chunk, and statistics and counters by device-scope
// accesses without cache-wide fences.  us a call (the sweep; this; with keys through registers, three barriers and fences):
// 32 heads x 128, 256 rows, 4k keys 30, 47, 90; 8k 42, 68, 125; 32k 131, 198, 353; 8 sequences x 8k, 512 rows 481, 773, 1892.
template <int D>
__device__ __forceinline__ void sweep_redo(const SweepParams& prm, uint32_t lds0) {
  using C = Cfg<D>;
  constexpr int S = C::kSteps;
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid), "+s"(lds0));  // (what is formed from them would be kept in registers for the whole of the walk)
  const int lane = tid & 63, r = lane & 31, g = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int spans = prm.spans, tasks = prm.B * prm.heads() * prm.nqg * spans, tasks2 = prm.B * prm.heads() * prm.spans2;  // of the two passes
  const uint32_t word = lds0 + C::kOffMass;                   // one int: the ticket, or whether to go on
  const uint32_t colsum = lds0 + C::kOffCs;                   // [2][kWaves][kKeys] floats
  for (;;) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (transfers of the last task that nothing has waited for)
    __syncthreads();
    if (tid == 0) *in_lds<int>(word) = __hip_atomic_fetch_add(&prm.ctl->ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const int ticket = __builtin_amdgcn_readfirstlane(*in_lds<int>(word));
    if (ticket >= tasks + tasks2) return;
    const bool second = ticket >= tasks;
    const int pieces = second ? prm.spans2 : spans;
    const int task = second ? ticket - tasks : ticket;
    const int span = task % pieces, first = second ? task / pieces * prm.nqg : task / pieces;  // (first unit)
    const int bh = first / prm.nqg;
    const int b = bh / prm.heads(), h = bh % prm.heads() / prm.subsets;
    const int P = prm.lens.P[b];
    const int nc = ceil_div(P, kKeys);
    const int c0 = nc * span / pieces, c1 = nc * (span + 1) / pieces;
    float head_mass = 0.f;
    for (int unit = first; unit < first + (second ? prm.nqg : 1); ++unit) {
      const char* area = prm.units + (int64_t)unit * kUnitBytes<D>;
      u32x4 qf[S];
#pragma unroll
      for (int s = 0; s < S; ++s) qf[s] = *reinterpret_cast<const u32x4*>(area + kRowsAt + wave * C::kQBytes + s * 1024 + lane * 16);
      float2* st = prm.stats + (int64_t)unit * spans * kRows + wave * 32 + r;  // (of query row r; one span is kRows further)
      float m = kNegBig, l = 0.f;
      float nl[16];  // second pass: minus the base-2 log-sum-exp of this lane's rows
      if (second) {
        if (tid == 0) {
          const uint64_t t0 = wall_clock64();
          while (__hip_atomic_load(&prm.spans_done[unit], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < spans && wall_clock64() - t0 < kTaskWait)
            __builtin_amdgcn_s_sleep(8);
        }
        asm volatile("" ::: "memory");
        __syncthreads();
        // all spans and the response span
        const float* refs = reinterpret_cast<const float*>(area + kRefsAt) + wave * 64 + r;
        const float ref = -refs[0] * prm.c;  // +inf for a row that does not exist
        const float own = refs[32];
        const bool live = ref != INFINITY;
        float M = live ? ref : 0.f, Lp = 0.f;
        float2 v[kSpans];
#pragma unroll
        for (int i = 0; i < kSpans; ++i) {
          v[i] = make_float2(kNegBig, 0.f);
          if (i < spans) {
            v[i].x = __hip_atomic_load(&st[i * kRows].x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            v[i].y = __hip_atomic_load(&st[i * kRows].y, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          }
          M = fmaxf(M, v[i].x);
        }
#pragma unroll
        for (int i = 0; i < kSpans; ++i) Lp += v[i].y * fast_exp2(v[i].x - M);
        const float L = fmaf(own, fast_exp2(ref - M), Lp);
        const float nlse = live ? -(M + __log2f(L)) : -INFINITY;
        if (span == 0 && prm.mass) {
          float mass = live && g == 0 ? Lp / L : 0.f;
#pragma unroll
          for (int o = 32; o > 0; o >>= 1) mass += __shfl_xor(mass, o, 64);
          if (lane == 0) *in_lds<float>(colsum + wave * 4) = mass;
          __syncthreads();
          if (tid == 0) {
            float t = 0.f;
            for (int w = 0; w < kWaves; ++w) t += *in_lds<float>(colsum + w * 4);
            head_mass += t;
            if (unit == first + prm.nqg - 1) prm.mass[bh] = head_mass;
          }
          __syncthreads();
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) nl[i] = __shfl(nlse, 8 * (i / 4) + 4 * g + (i % 4), 64);
      }
      auto dma = [&](int n) {  // chunk number n of the span (or its last one) into slot n of the ring
        const int ci = min(c0 + n, c1 - 1), last = P - 1 - ci * kKeys;
        const char* base = prm.K.row(b, h, ci * kKeys);
#pragma unroll
        for (int j = 0; j < C::kMoves; ++j) {
          const int row = wave * (kKeys / kWaves) + j * C::kRPI + lane / C::kPPR;
          const int piece = (lane % C::kPPR) ^ C::swz(row);
          dma16(base, (uint32_t)min(row, last) * (uint32_t)prm.K.stride_t + piece * 16,
                lds0 + n % C::kRing * C::kKBytes + (wave * (kKeys / kWaves) + j * C::kRPI) * C::kRowB);
        }
      };
      auto flush = [&](int n) {  // column sums of chunk n of the span
        const int j = (c0 + n) * kKeys + (int)tid;
        if ((int)tid >= kKeys || j >= P) return;
        const uint32_t cs = colsum + (n & 1) * kWaves * kKeys * 4 + tid * 4;
        float v = 0.f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) v += *in_lds<const float>(cs, w * kKeys * 4);
        // Whole sums only are stored: a workgroup that is still in its walk stores the same ones at any time, which would otherwise count
        // the groups before twice.
        const uint32_t kept = lds0 + C::kOffStart + (n * kKeys + tid) * 4;
        if (unit > first) v += *in_lds<const float>(kept);
        if (unit < first + prm.nqg - 1)
          *in_lds<float>(kept) = v;
        else
          __hip_atomic_store(prm.out + (int64_t)bh * prm.out_stride + j, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      };
      if (c0 < c1) {
        dma(0);
        dma(1);
      }
      auto walk = [&](auto columns) {  // a pass's instructions in a loop of their own
        constexpr bool kColumns = decltype(columns)::value;
        for (int n = 0; n < c1 - c0; ++n) {
          dma(n + 2);  // (its slot was last read before the barrier of the step before)
          asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"i"(2 * C::kMoves) : "memory");
          if (kColumns && n > 0) flush(n - 1);
          const uint32_t chunk = lds0 + n % C::kRing * C::kKBytes;
          f32x16 a[kNB];
#pragma unroll
          for (int kb = 0; kb < kNB; ++kb) {
            a[kb] = f32x16{};
#pragma unroll
            for (int s = 0; s < S; ++s) {
              const u32x4 kf = *in_lds<const u32x4>(chunk + (kb * 32 + r) * C::kRowB + (((2 * s + g) ^ C::swz(r)) << 4));
              if constexpr (kColumns)
                mfma_step<bf16_t>(qf[s], kf, a[kb]);
              else
                mfma_step<bf16_t>(kf, qf[s], a[kb]);
            }
          }
          if constexpr (kColumns) {
#pragma unroll
            for (int kb = 0; kb < kNB; ++kb) {
              float v = 0.f;
#pragma unroll
              for (int i = 0; i < 16; ++i) v += fast_exp2(fmaf(a[kb][i], prm.c, nl[i]));
              v = sum_halves(v);
              if (g == 0) *in_lds<float>(colsum + ((n & 1) * kWaves * kKeys + wave * kKeys + kb * 32 + r) * 4) = v;
            }
          } else {
            const int left = P - (c0 + n) * kKeys;
            if (left < kKeys)
#pragma unroll
              for (int kb = 0; kb < kNB; ++kb)
#pragma unroll
                for (int i = 0; i < 16; ++i)
                  if (kb * 32 + 8 * (i / 4) + 4 * g + (i % 4) >= left) a[kb][i] = -INFINITY;
            float top = a[0][0];
#pragma unroll
            for (int kb = 0; kb < kNB; ++kb)
#pragma unroll
              for (int i = 0; i < 16; ++i) top = fmaxf(top, a[kb][i]);
            const float bm = fmaxf(m, top * prm.c);
            float v = 0.f;
#pragma unroll
            for (int kb = 0; kb < kNB; ++kb)
#pragma unroll
              for (int i = 0; i < 16; ++i) v += fast_exp2(fmaf(a[kb][i], prm.c, -bm));
            l = l * fast_exp2(m - bm) + v;
            m = bm;
          }
        }
      };
      if (second)
        walk(std::true_type());
      else
        walk(std::false_type());
      if (second && c0 < c1) {
        __syncthreads();
        flush(c1 - c0 - 1);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (the next group's transfers reuse the ring)
        __syncthreads();
      }
      if (!second) {
        const float mo = xor32(m), lo = xor32(l);
        const float mm = fmaxf(m, mo);
        if (g == 0) {
          __hip_atomic_store(&st[span * kRows].x, mm, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          __hip_atomic_store(&st[span * kRows].y, l * fast_exp2(m - mm) + lo * fast_exp2(mo - mm), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        // (Device-scope stores that have completed are seen by every device-scope load that is issued later; a release here would
        // write back the whole L2, an acquire above throw it away.)
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (tid == 0) __hip_atomic_fetch_add(&prm.spans_done[unit], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
  }
}

// What a step of a walk works on: a chunk of a head's keys and one of the head's groups of voting rows.
struct Task {
  int bh, qg;
  uint32_t shape;
  uint32_t at;  // its unit's place in SweepParams::units
  __device__ bool idle() const { return shape == 0; }
  __device__ int ci() const { return shape & 255; }
  __device__ int nc() const { return (shape >> 8 & 255) + 1; }
  __device__ int keys() const { return shape >> 16; }
  __device__ int unit(const SweepParams& prm) const { return bh * prm.nqg + qg; }
};
// the chunk whose workgroup writes the head's mass (not always the first, so that they are spread over workgroups)
__device__ __forceinline__ int lead_of(int bh, int nc) { return (bh & 15) < nc ? bh & 15 : 0; }

// the row (of a wave's 32) whose sum the butterfly of `publish` leaves in a lane; lanes 2n and 2n+1 hold the same one
__device__ __forceinline__ int row_of(int ln) {
  return 8 * (((ln >> 4) & 1) * 2 + ((ln >> 3) & 1)) + 4 * (ln >> 5) + (((ln >> 2) & 1) * 2 + ((ln >> 1) & 1));
}

// After the walk: the masses of the heads whose leading chunk was this workgroup's and that have waves with mostly small row sums.  A head's
// mass is stored once and as a whole: the fallback of another workgroup may have stored it by now, and a part would take its place, or be
// added to it.
template <int D>
__device__ __forceinline__ void late_masses(const SweepParams& prm, uint32_t lds0, int next) {
  using C = Cfg<D>;
  int lane = threadIdx.x & 63;
  asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" : "+v"(lane) : : "memory");  // (this workgroup's own parts and its list are there)
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int unit = 0, units = 0;  // of the present head: the next one, and how many are left
  float mass = 0.f;
  while (next || units) {
    if (units == 0) {
      unit = (next - 1) * prm.nqg;
      units = prm.nqg;
      mass = 0.f;
      next = __builtin_amdgcn_readfirstlane(__hip_atomic_load(&prm.late[next - 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    }
    const int bh = unit / prm.nqg;
    const int nc = ceil_div(prm.lens.P[bh / prm.heads()], kKeys);
    const int lead = lead_of(bh, nc);
    const uint32_t* part = prm.parts + ((int64_t)unit * kWaves + wave) * prm.n_parts;
    const uint64_t t0 = wall_clock64();
    float sum = 0.f;
    while (wave * 32 < prm.rows) {
      uint32_t u[kMaxGroups / 64];
#pragma unroll
      for (int j = 0; j < kMaxGroups / 64; ++j) {
        u[j] = 0;
        if (j * 64 + lane < nc) u[j] = __hip_atomic_load(part + j * 64 + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      if (__all(__hip_atomic_load(part + lead, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == kNoPart)) {  // not one of those waves
        const uint64_t* low = reinterpret_cast<const uint64_t*>(prm.units + (int64_t)unit * kUnitBytes<D>) + wave * 32 + row_of(lane);
        uint64_t lo = 0;
#pragma unroll
        for (int j = 0; j < kCopies; ++j)
          lo += __hip_atomic_load(low + j * kRows, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint64_t hi = __hip_atomic_load(low + kCopies * kRows, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const float L = fmaf(whole(hi), 1.f / kHighScale, whole(lo) * (1.f / kLowScale));
        sum = lane % 2 ? 0.f : row_mass(L, reciprocal(L));
        break;
      }
      sum = 0.f;
      bool there = true;
#pragma unroll
      for (int j = 0; j < kMaxGroups / 64; ++j) {
        there = there && u[j] != kNoPart;
        sum += as_f32(u[j]);
      }
      if (__all(there)) break;
      if (wall_clock64() - t0 >= (uint64_t)prm.patience || __any(__hip_atomic_load(&prm.ctl->redo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))) {
        __hip_atomic_store(&prm.ctl->redo, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *in_lds<int>(lds0 + C::kOffBad) = 1;
        break;
      }
      __builtin_amdgcn_s_sleep(8);
    }
    sum = wave_sum(sum);
    if (lane == 0) *in_lds<float>(lds0 + C::kOffMass + wave * 4) = sum;
    __syncthreads();
    ++unit;
    --units;
    if (threadIdx.x == 0) {
      mass += sum_of_waves<kWaves>(lds0 + C::kOffMass);
      if (units == 0 && !*in_lds<const int>(lds0 + C::kOffBad)) __hip_atomic_store(&prm.mass[bh], mass, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
  }
}

// HALVES: a head has at most 128 voting rows, and each half of the workgroup works on chunks of its own, as a workgroup of four waves
// (with a ring of two chunks, and in the rounds without one on an idle task).
template <int D, bool HALVES>
__device__ __forceinline__ void sweep_chunks(const SweepParams& prm, uint32_t lds0) {
  using C = Cfg<D>;
  constexpr int S = C::kSteps;
  constexpr int kTeam = HALVES ? kWaves / 2 : kWaves;  // waves that share a chunk
  constexpr int kSlots = HALVES ? C::kRing / 2 : C::kRing;
  constexpr int kShare = kKeys / kTeam;                // keys that a wave moves
  constexpr int kMoves = kShare / C::kRPI;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane & 31, g = lane >> 5;
  const bool second = wave >= kWaves / 2;  // the group of waves that runs half a step behind
  const int rb = wave % kTeam;             // this wave's block of 32 rows
  const int lds_ring = lds0 + (HALVES && second ? kSlots * C::kKBytes : 0);
  const float c = prm.c;
  // A value hidden from the optimiser: what a step derives from it is then worth an instruction or two each time instead of
  // a register for the whole loop.
  auto here = [&](uint32_t v) {
    asm volatile("" : "+v"(v));
    return v;
  };
  auto lane_now = [&]() { return (int)here(lane); };

  // ---- the walk
  typedef const __attribute__((address_space(4))) Chunk* Table;
  const int team = (int)blockIdx.x + (HALVES && second ? (int)gridDim.x : 0);
  const Table table = (Table)(prm.table + (int64_t)team * prm.rounds);
  auto count = [&](int t) { return *(const __attribute__((address_space(4))) int*)(prm.counts + t); };
  const int chunks = HALVES && team >= prm.plan.groups ? 0 : count(team);
  const int mine = chunks * prm.nqg;  // steps: each chunk with all groups of voting rows, so that keys are transferred once
  const uint32_t kstride = (uint32_t)prm.K.stride_t;
  const uint32_t lane16 = lane * 16;
  // Row rb * kShare + j * kRPI + rl of the chunk (rl: this lane's row of transfer j) has its pieces permuted by the low bits of
  // that number, which are j's and rl's side by side: one exclusive-or with a constant per transfer.
  const uint32_t krow = (uint32_t)lane / C::kPPR, kpiece = ((uint32_t)lane % C::kPPR ^ C::swz(krow)) << 4;
  const uint32_t koff = (rb * kShare + krow) * kstride;  // (a chunk's rows are up to 127 x 16 MiB apart)
  // Chunk number t into its slot of the ring: this wave's part.  (Rows past the last key re-read it.)
  auto dma_keys = [&](int t, uint32_t shape, const char* keys) {
    const uint32_t most = (max(shape >> 16, 1u) - 1) * kstride;
    const uint32_t to = lds_ring + t % kSlots * C::kKBytes + rb * kShare * C::kRowB;
#pragma unroll
    for (int j = 0; j < kMoves; ++j)
      dma16(keys, min(here(koff) + (uint32_t)(j * C::kRPI) * kstride, most) + (here(kpiece) ^ (C::swz(j * C::kRPI) << 4)), to + j * 1024);
  };
  auto dma_k = [&](int t) {
    const Table c = table + min(t, chunks - 1);
    dma_keys(t, c->shape, c->keys);
  };
  const Base units = base_of(prm.units);
  auto dma_start = [&](const Task& k, int par) {
    dma4((const char*)units, (here(lane16) >> 2) + (k.at + kRefsAt + rb * 256), lds0 + C::kOffStart + (par * kWaves + wave) * 256);
  };
  u32x4 qf[S];
  // (The loads of the walk are asm, and waited for by asm: the compiler does not see the transfers and would wait for all of them.)
  uint32_t q_at = 0;
  auto aim_q = [&](const Task& k) { q_at = here(lane16) + (k.at + kRowsAt + rb * C::kQBytes); };
  auto load_q = [&](int ks) {
    if (ks == 4) q_at += 4096;  // (what an immediate offset reaches)
    asm volatile("global_load_dwordx4 %0, %1, %2 offset:%3" : "=v"(qf[ks]) : "v"(q_at), "s"(units), "i"(ks % 4 * 1024));
  };

  const uint32_t row8 = (rb * 32 + row_of(lane)) * 8;
  const int copy = team % kCopies;
  bool patient = true;

  // The logits are formed 32 keys at a time, minus the rows' references, which are the accumulators' initial values (a
  // key past the prompt starts from -inf).  Matrix and vector instructions are interleaved by hand, in slots of one
  // MFMA, the exponentials of 16 / S logits of the block before, and the LDS read of the fragment of the MFMA
  // two slots on: left to itself the compiler waits for every fragment and moves the exponentials out of the way.
  auto init = [&](int par, int kb, int left, f32x16& a) {
    const uint32_t nb = (left > kb * 32 ? lds0 + C::kOffStart + (par * kWaves + wave) * 256 : lds0 + C::kOffInf) + 16 * g;
#pragma unroll
    for (int i4 = 0; i4 < 4; ++i4) {
      const f32x4 v = *in_lds<const f32x4>(nb, 32 * i4);
#pragma unroll
      for (int e = 0; e < 4; ++e) a[4 * i4 + e] = v[e];
    }
  };
  uint32_t fa[S];  // this lane's fragments of the chunk
#pragma unroll
  for (int ks = 0; ks < S; ++ks) {
    fa[ks] = lds_ring + r * C::kRowB + (((2 * ks + g) ^ C::swz(r)) << 4);
    asm volatile("" : "+v"(fa[ks]));
  }
  int slot = 0;
  auto turn = [&]() {  // to the ring's next chunk
    const int by = slot == kSlots - 1 ? (1 - kSlots) * C::kKBytes : C::kKBytes;
    slot = slot == kSlots - 1 ? 0 : slot + 1;
#pragma unroll
    for (int ks = 0; ks < S; ++ks) fa[ks] += by;
  };
  u32x4 kf[kAhead + 1];
  auto fetch = [&](int n) {  // fragment n % S of block n / S
    kf[n % (kAhead + 1)] = *in_lds<const u32x4>(fa[n % S], n / S * 32 * C::kRowB);
  };
  float rs[16];
  constexpr int E = 16 / S;  // logits per slot
  float arg[E];
  // Slot m of the exponentials of a chunk: the arguments of the next slot's, this slot's exponentials, the sums of the last
  // slot's (three independent strands: a wave issues in order and would wait for each result in turn).
  auto expo = [&](int m, f32x16 (&p)[kNB]) {
    float v[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int i = m % S * E + e;
      if (m >= 0 && m < kNB * S) v[e] = fast_exp2(arg[e]);
      if (m + 1 >= 0 && m + 1 < kNB * S) {
        const int j = (m + 1) % S * E + e;
        arg[e] = p[(m + 1) / S][j] * c;
        asm volatile("" : "+v"(arg[e]));
      }
      if (m >= 1) {
        const int q = (m - 1) / S, j = (m - 1) % S * E + e;
        if (q > 0) {
          rs[j] = (q == 1 ? p[0][j] : rs[j]) + p[q][j];
          asm volatile("" : "+v"(rs[j]));
        }
      }
      if (m >= 0 && m < kNB * S) {
        asm volatile("" : "+v"(v[e]));
        p[m / S][i] = v[e];
      }
    }
  };

  // Column sums of a chunk that is completed for all groups of voting rows: add the waves' parts.  Four waves do it, 32 keys each;
  // the halves of a wave add half of the parts each.  (One store is issued in any case: vector() counts it.)  And the mass.
  const bool flushes = HALVES || !second;
  float mass = 0.f;  // of the head, as far as it is known
  int flushed = 0;   // chunks
  auto flush = [&](const Task& k, int par, bool there) {
    const int ln = lane_now();
    const int col = rb * 32 + (ln & 31);
    const uint32_t cs = lds0 + C::kOffCs + (par * kWaves + (HALVES && second ? kTeam : 0) + (ln >> 5) * (kTeam / 2)) * kKeys * 4 + col * 4;
    const int bad = *in_lds<const int>(lds0 + C::kOffBad);
    float v[kTeam / 2];
#pragma unroll
    for (int w = 0; w < kTeam / 2; ++w) v[w] = *in_lds<const float>(cs, w * kKeys * 4);
    const bool whole = k.qg == prm.nqg - 1;
    const int good = __builtin_amdgcn_readfirstlane(there && !(HALVES && k.idle()) ? bad ^ 1 : 0);
    const int keys = good && whole ? min(max(k.keys() - rb * 32, 0), 32) : 0;
    const uint32_t lanes = __builtin_amdgcn_readfirstlane((uint32_t)((1ull << keys) - 1));
    float t = v[0] + v[1];
    if (!HALVES) t += v[kTeam / 2 - 2] + v[kTeam / 2 - 1];
    const auto sw = __builtin_amdgcn_permlane32_swap(as_u32(t), as_u32(t), false, false);
    const unsigned u0 = sw[0], u1 = sw[1];
    t = as_f32(u0) + as_f32(u1);
    uint64_t exec;
    asm volatile("s_mov_b64 %0, exec\n\ts_mov_b64 exec, %1\n\tglobal_store_dword %2, %3, %4\n\ts_mov_b64 exec, %0"
                 : "=&s"(exec) : "s"((uint64_t)lanes), "v"(col * 4), "v"(t), "s"(table[flushed].out) : "memory");
    if (there && whole) ++flushed;
    if (rb == 0 && good && k.ci() == lead_of(k.bh, k.nc()) && prm.mass) {
      const uint32_t ms = lds0 + C::kOffMass + (par * kWaves + wave) * 4;
      const uint32_t late = lds0 + C::kOffLate + (HALVES && second ? 4 : 0);
      mass += sum_of_waves<kTeam>(ms);  // (below 0 from a mark on)
      if (whole) {
        if (__builtin_amdgcn_readfirstlane((int)as_u32(mass)) < 0) {  // (not known yet)
          if (ln == 0) {
            __hip_atomic_store(at<int>(base_of(prm.late + k.bh), here(0)), *in_lds<const int>(late), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            *in_lds<int>(late) = k.bh + 1;
          }
        } else if (ln == 0) {
          __hip_atomic_store(&prm.mass[k.bh], mass, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        mass = 0.f;
      }
    }
  };

  uint64_t seen[kCopies];
  auto ask = [&](const Task& k) {
    const uint32_t off = here(row8) + k.at;
#pragma unroll
    for (int i = 0; i < kCopies; ++i)
      asm volatile("global_load_dwordx2 %0, %1, %2 offset:%3 sc1" : "=v"(seen[i]) : "v"(off + i / 2 * 2 * kRows * 8), "s"(units), "i"(i % 2 * kRows * 8));
  };
  auto ask_again = [&](const Task& k) {
    const uint32_t off = here(row8) + k.at;
#pragma unroll
    for (int i = 0; i < kCopies; ++i) seen[i] = peek(units, off + i * kRows * 8);
    asm volatile("" ::: "memory");
  };
  auto add = [&](uint32_t at, float f, uint64_t lanes) {  // one chunk and the whole number next to f < 2^46, by these lanes
    f = rintf(f);
    const float top = floorf(f * 2.3283064365386963e-10f);  // 2^-32
    const uint32_t hi = (uint32_t)top + (1u << (kCountShift - 32));
    const uint32_t lo = (uint32_t)fmaf(top, -4294967296.f, f);
    const uint64_t v = ((uint64_t)hi << 32) | lo;
    uint64_t exec;
    asm volatile("s_mov_b64 %0, exec\n\ts_mov_b64 exec, %1\n\tglobal_atomic_add_x2 %2, %3, %4\n\ts_mov_b64 exec, %0"
                 : "=&s"(exec) : "s"(lanes), "v"(here(row8) + at), "v"(v), "s"(units) : "memory");
  };
  auto publish = [&](const Task& k) {  // this wave's row sums (rs) of the chunk just formed
    // sum over the 32 lanes of a half: 16 values, halved at every exchange
    float t8[8], t4[4], t2[2];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const auto sw = __builtin_amdgcn_permlane16_swap(as_u32(rs[i]), as_u32(rs[i + 8]), false, false);
      const unsigned u0 = sw[0], u1 = sw[1];
      t8[i] = as_f32(u0) + as_f32(u1);
    }
    // x + (x of the mirrored lane) in the lanes whose bit is clear, y + (y of the mirrored lane) in the others
    asm("s_nop 1\n\t"
        "v_add_f32_dpp %0, %4, %4 row_mirror row_mask:0xf bank_mask:0x3\n\tv_add_f32_dpp %1, %5, %5 row_mirror row_mask:0xf bank_mask:0x3\n\t"
        "v_add_f32_dpp %2, %6, %6 row_mirror row_mask:0xf bank_mask:0x3\n\tv_add_f32_dpp %3, %7, %7 row_mirror row_mask:0xf bank_mask:0x3\n\t"
        "v_add_f32_dpp %0, %8, %8 row_mirror row_mask:0xf bank_mask:0xc\n\tv_add_f32_dpp %1, %9, %9 row_mirror row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %2, %10, %10 row_mirror row_mask:0xf bank_mask:0xc\n\tv_add_f32_dpp %3, %11, %11 row_mirror row_mask:0xf bank_mask:0xc"
        : "=&v"(t4[0]), "=&v"(t4[1]), "=&v"(t4[2]), "=&v"(t4[3])
        : "v"(t8[0]), "v"(t8[1]), "v"(t8[2]), "v"(t8[3]), "v"(t8[4]), "v"(t8[5]), "v"(t8[6]), "v"(t8[7]));
    asm("s_nop 1\n\t"
        "v_add_f32_dpp %0, %2, %2 row_half_mirror row_mask:0xf bank_mask:0x5\n\tv_add_f32_dpp %1, %3, %3 row_half_mirror row_mask:0xf bank_mask:0x5\n\t"
        "v_add_f32_dpp %0, %4, %4 row_half_mirror row_mask:0xf bank_mask:0xa\n\tv_add_f32_dpp %1, %5, %5 row_half_mirror row_mask:0xf bank_mask:0xa"
        : "=&v"(t2[0]), "=&v"(t2[1]) : "v"(t4[0]), "v"(t4[1]), "v"(t4[2]), "v"(t4[3]));
    const int ln = lane_now();
    const float q0 = t2[0] + dpp<0x1B>(t2[0]), q1 = t2[1] + dpp<0x1B>(t2[1]);  // quad mirror
    float sum = (ln & 2) ? q1 : q0;
    sum += dpp<0xB1>(sum);  // neighbours
    const bool low = sum < kLowLimit;
    add(k.at + copy * kRows * 8, fminf(sum, kLowLimit) * kLowScale, HALVES && k.idle() ? 0 : __ballot(!(ln & 1) && low));
    if (!__all(low) && !(HALVES && k.idle())) {  // (rare)
      const bool fits = sum < kHighLimit;
      if (!__all(low || fits)) {  // known to every workgroup of the unit before its row sums are complete
        __hip_atomic_store(&prm.ctl->redo, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
      }
      add(k.at + kHighAt, fits ? sum * kHighScale : 0.f, __ballot(!(ln & 1) && !low));
    }
  };
  // Column sums of the chunk held in pc, once the row sums of its unit are all there, added to those of the groups before.
  float sums[kNB / 2] = {};
  auto complete = [&](const Task& k, int par, f32x16 (&pc)[kNB]) {
    uint64_t lo = 0, hi = 0;
#pragma unroll
    for (int i = 0; i < kCopies; ++i) lo += seen[i];
    bool ready = __all((int)(lo >> kCountShift) == k.nc());
    if (!ready && patient) {
      const uint64_t t0 = wall_clock64();
      do {
        __builtin_amdgcn_s_sleep(8);  // (a line that is asked for is slow to add to)
        ask_again(k);
        hi = peek(units, here(row8) + (k.at + kHighAt));
        lo = 0;
#pragma unroll
        for (int i = 0; i < kCopies; ++i) lo += seen[i];
        ready = __all((int)(lo >> kCountShift) + (int)(hi >> kCountShift) == k.nc());
      } while (!ready && wall_clock64() - t0 < (uint64_t)prm.patience);
      // Not every workgroup is running, or a row's sum is out of range: the scores of this workgroup are void from here on.
      if (!ready) {
        patient = false;
        __hip_atomic_store(&prm.ctl->redo, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      if (__any(hi != 0)) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
      if (!ready || (__any(hi != 0) && __hip_atomic_load(&prm.ctl->redo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)))
        *in_lds<int>(lds0 + C::kOffBad) = 1;
    }
    float L = whole(lo) * (1.f / kLowScale);
    if (__any(hi != 0)) L = fmaf(whole(hi), 1.f / kHighScale, L);
    const float w_row = reciprocal(L);
    *in_lds<float>(lds0 + C::kOffW + (HALVES && second ? kTeam * 128 : 0) + row8 / 2) = w_row;
    const bool small = mostly_small(L);
    if (k.ci() == lead_of(k.bh, k.nc())) {  // the mass of this wave's rows, or a mark that it is not known yet
      const int ln = lane_now();
      float ms = wave_sum((ln & 1) ? 0.f : row_mass(L, w_row));
      if (small) ms = -1e30f;
      if (ln == 0) *in_lds<float>(lds0 + C::kOffMass + (par * kWaves + wave) * 4) = ms;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    float w[16];
#pragma unroll
    for (int i4 = 0; i4 < 4; ++i4) {
      const f32x4 v = *in_lds<const f32x4>(lds0 + C::kOffW + wave * 128 + 16 * g, 32 * i4);
#pragma unroll
      for (int e = 0; e < 4; ++e) w[4 * i4 + e] = v[e];
    }
    float col[kNB];
#pragma unroll
    for (int kb = 0; kb < kNB; ++kb) {
      float a = 0.f, b = 0.f;
#pragma unroll
      for (int i = 0; i < 16; i += 2) {
        a = fmaf(pc[kb][i], w[i], a);
        b = fmaf(pc[kb][i + 1], w[i + 1], b);
      }
      col[kb] = a + b;
    }
    if (__builtin_expect(small, 0)) {
      const float t = wave_sum((col[0] + col[1]) + (col[2] + col[3]));
      if (lane_now() == 0)
        __hip_atomic_store(prm.parts + ((int64_t)k.unit(prm) * kWaves + rb) * prm.n_parts + k.ci(), as_u32(t) & 0x7FFFFFFFu, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    }
#pragma unroll
    for (int j = 0; j < kNB; j += 2) {  // lanes below 32 get block j, the others block j+1
      const auto sw = __builtin_amdgcn_permlane32_swap(as_u32(col[j]), as_u32(col[j + 1]), false, false);
      const unsigned u0 = sw[0], u1 = sw[1];
      sums[j / 2] += as_f32(u0) + as_f32(u1);
    }
    if (k.qg == prm.nqg - 1) {
      const uint32_t cs = lds0 + C::kOffCs + (par * kWaves + wave) * kKeys * 4 + lane16 / 4;
#pragma unroll
      for (int j = 0; j < kNB / 2; ++j) {
        *in_lds<float>(cs, j * 256) = sums[j];
        sums[j] = 0.f;
      }
    }
  };

  // ---- prologue: the first two chunks' keys, the first two steps' references and the first one's rows, then the third chunk's keys
  // (HALVES: the ring holds two chunks; a half without chunks asks for nothing)
  int fresh = 0;  // number of the chunk of `ahead`
  Task ahead{0, 0, 0, 0};
  auto take = [&](int bh, uint32_t shape) {
    ahead.bh = bh;
    ahead.shape = shape;
    ahead.at = (uint32_t)(bh * prm.nqg) * kUnitBytes<D>;
  };
  auto advance = [&]() {  // `ahead` to the walk's next task (which at the end of the walk may be of its last chunk again)
    ahead.at += kUnitBytes<D>;
    if (++ahead.qg < prm.nqg) return;
    ahead.qg = 0;
    const Table c = table + min(++fresh, chunks - 1);
    take(c->bh, c->shape);
  };
  // The first of a single sequence's chunks is where the plan has it, which is known before the table
  // is there; all that is asked for here is asked for before anything is waited for.  (One latency of a load that misses L2, of three: the
  // lock's word, the table, keys and rows.  4 to 16 rounds, us a call: 16 heads x 89 rows x 9.7k keys 25.5 -> 24.1, x 203 x 28k 59.6 ->
  // 58.5, 32 heads x 256 rows x 8k 37.2 -> 36.6, x 32k 115.5 -> 113.6, 4 heads x 1792 x 30k 89.8 -> 87.4.)
  const int run = *(const __attribute__((address_space(4))) int*)&prm.ctl->run;
  const int redo = *(const __attribute__((address_space(4))) int*)&prm.ctl->redo;
  uint32_t shape0 = 0;
  const char* keys0 = nullptr;
  const int run0 = HALVES && second && prm.plan.place(1) > 0 ? 1 : 0;
  if (prm.B == 1 && prm.plan.has(run0, team)) {
    const int P = prm.lens.P[0], nc = (P + kKeys - 1) / kKeys, off = team - prm.plan.place(run0);
    const int nth = off / nc, ci = off - nth * nc, vh = prm.plan.head(run0) + nth;
    take(vh, (uint32_t)ci | (uint32_t)(nc - 1) << 8 | (uint32_t)min(P - ci * kKeys, kKeys) << 16);
    shape0 = ahead.shape;
    keys0 = prm.K.row(0, prm.subsets == 1 ? vh : vh / prm.subsets, (int64_t)ci * kKeys);
  } else if (!HALVES || chunks > 0) {
    take(table->bh, table->shape);
    shape0 = table->shape;
    keys0 = table->keys;
  }
  Task cur = ahead, next = ahead, prev = ahead, done = ahead;
  uint32_t shape2 = 0;
  const char* keys2 = nullptr;
  if (!HALVES || chunks > 0) {
    dma_start(cur, 0);
    dma_keys(0, shape0, keys0);
    aim_q(cur);
#pragma unroll
    for (int ks = 0; ks < S; ++ks) load_q(ks);
    advance();
    next = ahead;
    dma_start(next, 1);
    dma_k(1);
    advance();
    const Table c = table + min(2, chunks - 1);
    shape2 = c->shape;
    keys2 = c->keys;
  }
  if (run && threadIdx.x == 0)
    __hip_atomic_fetch_add(&sweep_placed[blockIdx.x % kPlaces * kPlaceWords], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (threadIdx.x < 32) *in_lds<float>(lds0 + C::kOffInf + threadIdx.x * 4) = -INFINITY;
  // (kOffBad, kOffLate and kOffRedo; a workgroup that is placed when others have already given up, or that may not run as a sweep's, goes straight to
  // the fallback; what one wave has read of `redo` holds for all)
  if (threadIdx.x < 4) *in_lds<int>(lds0 + C::kOffBad + threadIdx.x * 4) = threadIdx.x == 0 ? redo : 0;
  for (int i = threadIdx.x; i < 2 * kWaves * kKeys; i += kThreads) *in_lds<float>(lds0 + C::kOffCs + i * 4) = 0.f;
  if (threadIdx.x < 2 * kWaves) *in_lds<float>(lds0 + C::kOffMass + threadIdx.x * 4) = 0.f;
  // (all but the second chunk's keys: each group of waves waits for its part of them before the other one forms that chunk, see below)
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"i"(1 + kMoves) : "memory");
#pragma unroll
  for (int ks = 0; ks < S; ++ks) asm volatile("" : "+v"(qf[ks]));
  if (__builtin_amdgcn_readfirstlane(*in_lds<const int>(lds0 + C::kOffBad))) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (no transfer into LDS outlives its workgroup, or meets the fallback's)
    return;
  }
  if (!HALVES) dma_keys(2, shape2, keys2);
  int keys_at = HALVES ? 2 : 3;  // number of the next chunk whose keys are asked for
  f32x16 pa[kNB], pb[kNB];
#pragma unroll
  for (int kb = 0; kb < kNB; ++kb) {
    pa[kb] = f32x16{};
    pb[kb] = f32x16{};
  }
  __builtin_amdgcn_sched_barrier(0);
  auto end_matrix = [&](int s) {
    __builtin_amdgcn_sched_barrier(0);
    if (s == 0 && mine > 16)  // (what was asked for so far, at once: 32k keys 113 us, 116 without; short walks lose by it)
      asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
    else
      asm volatile("s_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  auto end_vector = [&]() {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  auto shift = [&]() {
    done = prev;
    prev = cur;
    cur = next;
    next = ahead;
    advance();
  };
  // The first group forms the second chunk between this group's matrix and vector phase of the first, i.e. before this group has waited
  // for anything else: its part of that chunk's keys has to be there by now (the third's, kMoves transfers, may be in flight).  It costs
  // nothing, as the barrier is a matrix phase of the first group away.  (That group's part is waited for in its first vector phase, which
  // ends before this group forms the second chunk; halves move their own keys.)
  if (second) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"i"(kMoves) : "memory");

  if (HALVES && mine == 0) {  // no such half is in any round: it only meets the other's barriers
    for (int s = 0; s < count(team - (int)gridDim.x); ++s) {
      end_vector();
      end_vector();
    }
    end_vector();
    if (!second) end_vector();
    return;
  }
  // (Every workgroup that is launched has a step in some round, see Packing.  `for` loops, with that assumed for the compiler, took 146.1 us
  // for the 32k layer and 480 for the ragged scoring, these 144.9 and 477.)
  if (rb * 32 >= prm.rows) {  // no rows for this wave: it only helps to move keys and to add columns
    int s = 0;
    do {
      end_matrix(s);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      if (cur.qg == 0 && keys_at < chunks) dma_k(keys_at++);
      if (flushes) flush(done, s & 1 ^ 1, s >= 2);
      shift();
      end_vector();
    } while (++s < mine);
    end_vector();
    if (flushes) flush(done, mine & 1 ^ 1, mine >= 2);
    if (HALVES) flush(prev, mine & 1, true);
    if (!second) {
      end_vector();
      if (!HALVES) flush(prev, mine & 1, true);
    }
    return;
  }

  // Step s, matrix phase: chunk s is formed into pf; the rows of step s+1 are asked for as soon as their registers are free, then
  // the row sums of step s-1 (as late as an answer can be hidden: a sum that is asked for too early has to be asked for twice).
  auto matrix = [&](int par, f32x16 (&pf)[kNB]) {
    const int left = cur.keys() - r;  // keys of the chunk from this lane's on
#pragma unroll
    for (int i = 0; i < kAhead; ++i) fetch(i);
    init(par, 0, left, pf[0]);
#pragma unroll
    for (int n = 0; n < kNB * S; ++n) {
      const int kb = n / S, ks = n % S;
      if (n + kAhead < kNB * S) fetch(n + kAhead);
      if (ks == S / 2 && kb + 1 < kNB) init(par, kb + 1, left, pf[kb + 1]);
      mfma_step<bf16_t>(qf[ks], kf[n % (kAhead + 1)], pf[kb]);
      expo(n - S - kLag, pf);
      if (n == (kNB - 1) * S) aim_q(next);
      if (kb == kNB - 1) load_q(ks);
      __builtin_amdgcn_sched_barrier(0);
    }
    ask(prev);
    if (cur.qg == prm.nqg - 1) turn();
#pragma unroll
    for (int m = kNB * S - S - kLag; m <= kNB * S; ++m) expo(m, pf);
  };
  // Vector phase: the row sums published; step s-1, held in pc, is completed; the keys of the chunk after the next two and the
  // references of step s+2 are asked for.
  auto vector = [&](int s, int par, f32x16 (&pc)[kNB]) {
    publish(cur);
    if (flushes) flush(done, par ^ 1, s >= 2);
    // All but the addition and the store just issued: the rows, the row sums, and the transfers of the step before.
    if (!flushes)
      asm volatile("s_waitcnt vmcnt(1)" ::: "memory");
    else
      asm volatile("s_waitcnt vmcnt(2)" ::: "memory");
#pragma unroll
    for (int i = 0; i < kCopies; ++i) asm volatile("" : "+v"(seen[i]));
#pragma unroll
    for (int ks = 0; ks < S; ++ks) asm volatile("" : "+v"(qf[ks]));
    dma_start(ahead, par);
    if (s > 0 && !(HALVES && prev.idle())) complete(prev, par, pc);
    if (cur.qg == 0 && keys_at < chunks) dma_k(keys_at++);
    shift();
  };
  auto step = [&](int s, int par, f32x16 (&pf)[kNB], f32x16 (&pc)[kNB]) {
    matrix(par, pf);
    end_matrix(s);
    vector(s, par, pc);
    end_vector();
  };
  int s = 0;
  do {
    step(s, 0, pa, pb);
    if (s + 1 < mine) step(s + 1, 1, pb, pa);
    s += 2;
  } while (s < mine);
  // ---- the last step: completed at once, by the first group while the second publishes it
  const int par = mine & 1;
  // Whether others have given up, for the kernel's end (who gives up itself has kOffBad): by one wave for all of them, who have to agree,
  // and here, where its answer comes with those of the sums.
  int others = 0;
  if (wave == 0) others = __hip_atomic_load(&prm.ctl->redo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (!HALVES || !prev.idle()) {
    ask_again(prev);
    if (par)
      complete(prev, par, pa);
    else
      complete(prev, par, pb);
  }
  if (wave == 0 && lane == 0) *in_lds<int>(lds0 + C::kOffRedo) = others;
  end_vector();
  if (flushes) flush(done, par ^ 1, mine >= 2);
  if (HALVES) flush(prev, par, true);
  if (!second) {
    end_vector();
    if (!HALVES) flush(prev, par, true);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (no transfer into LDS outlives its workgroup)
}

// The kernel's argument, from a pointer hidden from the optimiser: what follows the walk then loads what it needs when it needs it,
// instead of having it loaded before the walk and kept in registers, or spilled, for the whole of it.
__device__ __forceinline__ const SweepParams& argument_again() {
  typedef const __attribute__((address_space(4))) SweepParams* Arg;
  Arg p = (Arg)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(const SweepParams*)p;
}

template <int D, bool HALVES>
__global__ __launch_bounds__(kThreads, 2) void sweep_kernel(const SweepParams prm) {
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;
  sweep_chunks<D, HALVES>(prm, lds0);
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  const int late = __builtin_amdgcn_readfirstlane(*in_lds<const int>(lds0 + Cfg<D>::kOffLate));
  const int late2 = HALVES ? __builtin_amdgcn_readfirstlane(*in_lds<const int>(lds0 + Cfg<D>::kOffLate, 4)) : 0;
  if (__builtin_expect(late, 0)) late_masses<D>(argument_again(), lds0, late);
  if (HALVES && __builtin_expect(late2, 0)) late_masses<D>(argument_again(), lds0, late2);
  const int redo = *in_lds<const int>(lds0 + Cfg<D>::kOffBad) | *in_lds<const int>(lds0 + Cfg<D>::kOffRedo);
  if (__builtin_amdgcn_readfirstlane(redo)) sweep_redo<D>(argument_again(), lds0);
}

__global__ void hold_kernel(int64_t age) {
  const uint32_t there = placed();
  const uint32_t then = (uint32_t)((wall_clock64() - (age < 0 ? 0 : (uint64_t)age)) >> kTick);
  if (threadIdx.x == 0) sweep_lock = ((unsigned long long)then << 32) | (there + (age < 0 ? 0 : kMaxGroups));
}

int cus() {
  static int n = 0;
  if (!n) {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) == hipSuccess && hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess) n = v;
    if (n < 1) n = 256;
  }
  return n;
}

size_t pad256(size_t n) { return (n + 255) / 256 * 256; }

// Pieces of a unit's keys in the fallback's first pass: two tasks for every compute unit, since a task costs about as much as two
// chunks before its first one.
int spans_of(int units) { return max(1, min(kSpans, 2 * kMaxGroups / units)); }

struct Layout {
  size_t control, table, counts, mass, done, late, parts, units, stats, bytes;  // offsets from the start of the area
  int n_parts;
  Layout(const maskkv_desc* d, int nqg, const SweepPlan& plan) {
    const size_t n = (size_t)d->B * d->H * nqg;  // units
    control = 0;
    table = pad256(sizeof(Control));
    counts = table + (size_t)plan.groups * plan.rounds * sizeof(Chunk);
    mass = counts + plan.groups * sizeof(int);
    done = mass + n * sizeof(float);
    n_parts = (d->P_max + kKeys - 1) / kKeys;
    late = done + n * sizeof(int);
    parts = late + n * sizeof(int);
    units = pad256(parts + n * kWaves * n_parts * sizeof(uint32_t));
    stats = units + n * (d->d == 128 ? kUnitBytes<128> : kUnitBytes<64>);
    bytes = stats + n * spans_of((int)n) * kRows * sizeof(float2);
  }
};

// How a description would be swept, and whether that is faster than the two passes.
//
// At most one workgroup per compute unit, since all have to be resident.  The workgroups of a head (one a chunk) wait for each
// other, so they work on it at the same time: a round puts as many heads side by side as there are workgroups for, the longest
// first, and is repeated for the next heads of the same sequences as long as these last.  (Dealt out end to end, heads straddle
// two rounds, and the first workgroups of such a head wait for the last: 503 instead of 481 us for the ragged batch, whose 18112
// chunks take 74 rounds of 256 workgroups instead of 71.)  Many sequences can make more runs than the plan has room for; each
// sequence then has rounds of its own.
//
// A head's groups of voting rows are one workgroup's turn, which needs its keys once, unless that leaves workgroups without work: a
// head then counts as several with the same keys, and their column sums are added by a kernel of their own (5 us).
//
// Where no head has more than 128 voting rows, four of a workgroup's waves would have none: the halves of a workgroup can then be two
// workgroups, each with chunks of its own (4 sequences of 28 heads, head_dim 64, 116 rows, 22 chunks: 37.6 instead of 44.9 us).
// The first halves and the second halves are packed by themselves (`half` workgroups each) unless a head on both saves enough.
// The halves meet at each step's barriers, so a step has the same number as its round in every half, and a half that a round
// has no chunk for goes through an idle step: with the steps of a list closed up, one half waits for a head of a later round
// than the other's, and halves that hold each other up this way can wait in a circle.
struct Packing {
  SweepPlan plan;
  int across = 0;  // of a head that lies on either side of `edge`, the chunks beyond it (the most of all rounds)
  Packing(const maskkv_desc* d, const int* nc, int n, int half, int edge, int subsets, bool mixed) : plan{} {
    int left[MASKKV_MAX_BATCH], order[MASKKV_MAX_BATCH], B = 0;
    for (int b = 0; b < d->B; ++b) {
      left[b] = nc[b] > 0 ? d->H * subsets : 0;
      if (left[b] == 0) continue;
      int i = B++;
      for (; i > 0 && nc[order[i - 1]] < nc[b]; --i) order[i] = order[i - 1];
      order[i] = b;
    }
    plan.subsets = subsets;
    for (int first = 0; first < B;) {
      if (left[order[first]] == 0) {
        ++first;
        continue;
      }
      const int run = plan.runs;
      int side_of[MASKKV_MAX_BATCH] = {};  // heads of a sequence in the round
      for (int from = 0; from < n; from += half) {
        int room = half;
        for (int i = first; i < (mixed ? B : first + 1) && room > 0; ++i) {
          const int b = order[i], side = min(left[b] - side_of[b], room / nc[b]);
          if (side == 0) continue;
          if (plan.runs == kMaxRuns) {
            plan.groups = 0;
            return;
          }
          const int at = from + half - room;
          plan.put(plan.runs++, at, side, side * nc[b], b, 0);
          if (at < edge && edge < at + side * nc[b] && (edge - at) % nc[b]) across = max(across, nc[b] - (edge - at) % nc[b]);
          room -= side * nc[b];
          side_of[b] += side;
          plan.groups = max(plan.groups, from + half - room);
        }
      }
      int times = 0x7FFFFFFF;
      for (int i = run; i < plan.runs; ++i) times = min(times, left[plan.sequence(i)] / side_of[plan.sequence(i)]);
      for (int i = run; i < plan.runs; ++i) {
        const int b = plan.sequence(i), side = plan.side(i);
        plan.put(i, plan.place(i), side, plan.width(i), b, d->H * subsets - left[b]);
        plan.repeat(i, times);
        left[b] -= side * times;
      }
      plan.rounds += times;
    }
  }
};

SweepPlan make_plan(const maskkv_desc* d, const Lens& lens, int nqg) {
  const int n = min(cus(), kMaxGroups);
  SweepPlan best{};
  int nc[MASKKV_MAX_BATCH], most = 0;
  int64_t chunks = 0;
  for (int b = 0; b < d->B; ++b) {
    nc[b] = (lens.P[b] + kKeys - 1) / kKeys;
    most = max(most, nc[b]);
    chunks += (int64_t)nc[b] * d->H;
  }
  if (most == 0 || most > n) return best;
  // Microseconds, from 70 batches of the sizes that bf16 prompts come in, each timed in every way: what a call costs besides its steps,
  // a step (256 rows; with half of the waves idle; of two chunks side by side), two passes per chunk.  (Rounds against two
  // passes, head_dim 128: 16 heads of 218 chunks 59 / 79, of 227 with two groups of rows 92 / 143, the 5952 chunks of 5 sequences
  // with 7 queries a head 88 / 131; head_dim 64: 28 heads of 213 chunks with two groups of rows 128 / 154, 1300 chunks 30 / 51.
  // Rounds against halves, head_dim 128: 32 heads of 87 chunks, 16 steps against 8, 43.6 / 38.3; 28 of 211, 28 / 14, 68.6 / 61; 16
  // of 163, 16 / 8, 46.6 / 41.3; but 8 of 163, 8 / 4, 29.7 / 30.0; 8 of 235, 8 / 4, 31.9 / 35.9; 28 of 39, 5 / 3, 22.4 / 22.9.)
  // A head on both halves of workgroups waits for the later one at every step, the longer the more of its chunks are there, but can
  // save rounds: 8 heads of 131 chunks, 6 across, 3 rounds against 4, 23.6 / 28.6; 32 of 87, 5 across, 7 / 8, 35.3 / 38.3; but
  // 8 of 163, 70 across, 3 / 4, 32.8 / 30.0; 28 of 211, 166 across, as many rounds, 115 / 61.
  const bool wide = d->d == 128, few = (int64_t)d->n_query * query_heads_per_kv(d) <= kRows / 2;
  double cost = 23.0 + (double)chunks * nqg * (wide ? 0.0169 : 0.0101);
  auto consider = [&](int workgroups, int half, int subsets, double besides, double step) {
    Packing p(d, nc, workgroups, half, n, subsets, true);
    if (!p.plan.groups) p = Packing(d, nc, workgroups, half, n, subsets, false);
    if (!p.plan.groups) return;
    p.plan.grid = min(p.plan.groups, n);
    const double c = besides + p.plan.rounds * ((nqg / subsets) * step + 0.02 * p.across);
    if (c >= cost) return;
    cost = c;
    best = p.plan;
  };
  for (int subsets = 1; subsets <= nqg; ++subsets)
    if (nqg % subsets == 0)
      consider(n, n, subsets, few ? (wide ? 12.4 : 10.6) : subsets > 1 ? 19.0 : 14.0, few ? (wide ? 2.07 : 1.87) : (wide ? 2.5 : 2.1));
  if (few)
    for (int half = n; half <= 2 * n; half += n) consider(2 * n, half, 1, wide ? 12.9 + 0.039 * most : 10.5 + 0.02 * most, wide ? 2.92 : 2.4);
  return best;
}

template <int D>
int launch(const maskkv_desc* d, const SweepParams& prm, hipStream_t stream) {
  const int lds_start = 2 * Cfg<D>::kKBytes, lds_start2 = lds_start + 2 * Cfg<D>::kQBytes;
  static bool raised = false;
  if (!raised) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&sweep_kernel<D, false>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, Cfg<D>::kLds);
    if (e == hipSuccess)
      e = hipFuncSetAttribute(reinterpret_cast<const void*>(&sweep_kernel<D, true>), hipFuncAttributeMaxDynamicSharedMemorySize,
                              Cfg<D>::kLds);
    if (e == hipSuccess)
      e = hipFuncSetAttribute(reinterpret_cast<const void*>(&sweep_start_kernel<D, 8>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, lds_start);
    if (e == hipSuccess)
      e = hipFuncSetAttribute(reinterpret_cast<const void*>(&sweep_start_kernel<D, 2>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, lds_start2);
    if (e != hipSuccess) {
      set_error("score: cannot raise dynamic LDS limit: %s", hipGetErrorString(e));
      (void)hipGetLastError();
      return MASKKV_EHIP;
    }
    raised = true;
  }
  const int units = prm.B * prm.H * prm.subsets * prm.nqg;
  if (units >= 128)
    hipLaunchKernelGGL((sweep_start_kernel<D, 8>), dim3(1 + prm.tables + units), dim3(kThreads), lds_start, stream, prm);
  else
    hipLaunchKernelGGL((sweep_start_kernel<D, 2>), dim3(1 + prm.tables + units * 4), dim3(kThreads), lds_start2, stream, prm);
  if (int e = check_launch("score (sweep start)")) return e;
  if (prm.plan.groups > prm.plan.grid)
    hipLaunchKernelGGL((sweep_kernel<D, true>), dim3(prm.plan.grid), dim3(kThreads), Cfg<D>::kLds, stream, prm);
  else
    hipLaunchKernelGGL((sweep_kernel<D, false>), dim3(prm.plan.grid), dim3(kThreads), Cfg<D>::kLds, stream, prm);
  return check_launch("score (sweep)");
}

}  // namespace

// A launch of 66000 units (33000 heads of 40 keys, 300 voting rows), once tried, ended in a memory fault whose cause was not found.
// The sweep is kept to the sizes that are in use (64 sequences x 32 heads x 2 groups of voting rows); more take the two passes.  (A
// unit's place in the workspace is held in 32 bits as well, which 55189 units of head_dim 128 would not fit.)
SweepPlan sweep_plan(const maskkv_desc* d, const Lens& lens, int nqg) {
  if (d->dtype != MASKKV_BF16 || (int64_t)d->B * d->H * nqg > kMaxUnits) return SweepPlan{};
  return make_plan(d, lens, nqg);
}

int hold_sweep(int64_t age_us, hipStream_t stream) {
  hipLaunchKernelGGL(hold_kernel, dim3(1), dim3(64), 0, stream, age_us < 0 ? -1 : age_us * 100);
  return check_launch("hold sweep");
}

size_t sweep_workspace_bytes(const maskkv_desc* d, int nqg, const SweepPlan& plan) { return Layout(d, nqg, plan).bytes; }

int launch_sweep(const maskkv_desc* d, const View& Q, const View& K, const Lens& lens, float scale, float* scores,
                 int64_t score_stride, float* prompt_mass, float* group_sums, int64_t group_stride, int nqg, const SweepPlan& plan,
                 void* area, hipStream_t stream, float** unit_mass) {
  SweepParams prm;
  prm.Q = Q;
  prm.K = K;
  prm.lens = lens;
  prm.B = d->B;
  prm.H = d->H;
  prm.n_resp = d->n_resp;
  prm.q_per_kv = query_heads_per_kv(d);
  prm.n_qh = d->n_query;
  prm.n_query = d->n_query * prm.q_per_kv;
  prm.subsets = plan.subsets;
  prm.nqg = nqg / plan.subsets;
  prm.rows = ((prm.n_query + nqg - 1) / nqg + 31) / 32 * 32;  // (as even as they can be: 300 rows are 160 and 140)
  prm.plan = plan;
  int64_t x = 0;  // steps of all workgroups
  for (int b = 0; b < d->B; ++b) x += (int64_t)((lens.P[b] + kKeys - 1) / kKeys) * d->H * nqg;
  // 100 us and about what the sweep takes, in which the fallback would be done, too.  (What keeps workgroups from being placed is
  // another program's kernels, a sweep of another process among them, whose lock is its own, or of another stream: the time
  // these take has nothing to do with this call's.  Two processes that score 32k keys at once, us a call of each: 455, with 20 ms 5000.)
  prm.patience = 10000 + (int)min(x / plan.groups * 500, (int64_t)1000000);
  prm.spans = spans_of(d->B * d->H * nqg);
  prm.spans2 = max(1, min(kMaxGroups, 2 * kMaxGroups / (d->B * d->H * plan.subsets)));
  if (prm.nqg > 1) prm.spans2 = max(prm.spans2, ((d->P_max + kKeys - 1) / kKeys + kSpanChunks - 1) / kSpanChunks);
  prm.c = scale * kLog2e;
  const Layout l(d, nqg, plan);
  char* base = reinterpret_cast<char*>(area);
  prm.ctl = reinterpret_cast<Control*>(base + l.control);
  prm.table = reinterpret_cast<Chunk*>(base + l.table);
  prm.counts = reinterpret_cast<int*>(base + l.counts);
  prm.tables = (d->B * d->H * plan.subsets + kWaves - 1) / kWaves;
  prm.rounds = plan.rounds;
  prm.spans_done = reinterpret_cast<int*>(base + l.done);
  prm.parts = reinterpret_cast<uint32_t*>(base + l.parts);
  prm.n_parts = l.n_parts;
  prm.late = reinterpret_cast<int*>(base + l.late);
  prm.stats = reinterpret_cast<float2*>(base + l.stats);
  prm.units = base + l.units;
  prm.out = plan.subsets == 1 ? scores : group_sums;
  prm.out_stride = plan.subsets == 1 ? score_stride : group_stride;
  prm.mass = plan.subsets == 1 ? prompt_mass : reinterpret_cast<float*>(base + l.mass);
  *unit_mass = plan.subsets == 1 ? nullptr : prm.mass;
  return d->d == 128 ? launch<128>(d, prm, stream) : launch<64>(d, prm, stream);
}

}  // namespace maskkv
