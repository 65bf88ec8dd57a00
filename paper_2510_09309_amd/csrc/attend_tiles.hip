// Tiled attention for bf16: one workgroup of eight waves serves 256 queries of one (b, h), 32 a wave, over 64-key tiles.
//
// The layout of the products is that of attend.hip (logits transposed, a lane owns one query, its probabilities are the B
// operand of O^T = V^T P^T).  What differs is how the three pipes of a SIMD are kept busy at the same time:
//
//   - K and V tiles come by direct transfers into two rings of four LDS slots, three tiles ahead, and no register or vector
//     instruction touches them on the way.  V stays row-major; the A operand V^T is read with transposing LDS loads.
//   - Waves 0-3 and 4-7 (one of each on a SIMD) run half a tile apart.  A tile is a matrix phase (its logits, and the output
//     update of the tile before) and a vector phase (its softmax).  One barrier a tile keeps one group of waves in the one while the
//     other is in the other: between barriers t and t+1 group 0 has the matrix phase of tile t and then its vector phase, group 1 the
//     vector phase of tile t-1 and then the matrix phase of tile t.
//
// The transfers K(t+3), V(t+2) ("pair t+3") are issued at the start of the vector phase of tile t; their slots were last read in
// matrix phases t-1 (K(t-1), V(t-2)), which both groups have left behind barrier t.
//
// Where 256 queries a workgroup leave compute units idle (HALVES), a workgroup serves 128: both groups have the same queries, group
// i takes tiles 2u + i through rings of two slots of its own, and the two partial results are merged through LDS, half by each group.
//
// What bounds it: power, in a loop of nothing but these calls, and before that the vector phase.  A tile of 256 queries takes 2880 cycles
// in the un-evicted call and 3200 in the short walks of a ragged batch (2048 of them MFMAs: a matrix phase is 1210 to 1250 cycles, a vector
// phase 230 to 410 for the transfers and 1140 to 1220 for the softmax, the rest waits); an earlier copy with counters gave 3150, and 3850 with
// the transfers' bases, strides and cases formed anew for each tile (690 cycles) and a barrier after every phase (the matrix phase's
// group waited 750 cycles for the other at each).  That is 18 % fewer cycles, of which the clock takes back three quarters: 33024 keys x 32 heads x
// 256 queries (head_dim 128), un-evicted call with its merge, 164 -> 157 us; eight sequences x 32 heads x 512 queries over 576 ... 1536
// keys (33 tiles on the busiest compute unit, 28 on average) 77.4 -> 74.4.  (The steps one by one: transfers 158 and 74.9, one barrier a tile
// 157 and 74.4.)  Not better: transfers between the MFMAs of the matrix phase (74.9 -> 77.3), five or seven fragments ahead (1 % in the former, nothing in
// the latter), even and odd waves as groups (both of a SIMD in the same phase), raised wave priority in the matrix phase.
#include <type_traits>

#include "attend.hpp"
#include "lds.hpp"

namespace maskkv {

namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int kWaves = 8;
constexpr int kTK = 64;      // keys per tile

template <int D, bool HALVES>
struct TileCfg {
  static constexpr int kQueries = HALVES ? 128 : 256;  // per workgroup
  static constexpr int kMovers = HALVES ? 4 : 8;       // waves that move a tile
  static constexpr int kMoveRows = kTK / kMovers;
  static constexpr int kRowB = D * 2;
  static constexpr int kSteps = D / 16;
  static constexpr int kDB = D / 32;
  static constexpr int kPPR = kRowB / 16;           // 16-byte pieces per row
  static constexpr int kRPI = 1024 / kRowB;         // rows moved by one wave instruction
  static constexpr int kMoves = kMoveRows / kRPI;   // transfers per wave and tile of K (and of V)
  static constexpr int kTileB = kTK * kRowB;
  static constexpr int kOffQ = 6 * kTileB;          // at first the queries, from the third V tile on (256 of them)
  static constexpr int kLds = (HALVES ? 8 : 10) * kTileB;  // four K tiles, four V tiles and, with 256 queries, room for the last of these
  static constexpr int kQK = 2 * kSteps;            // MFMAs of a tile's logits
  static constexpr int kPV = 4 * kDB;               // MFMAs of a tile's output update
  // A direct transfer writes 1 KiB of consecutive LDS, so rows carry no padding; instead a row's pieces are permuted.
  // K: piece p sits in slot p ^ swz_k(row): 16 consecutive rows of a fragment read fall on different 16-byte columns.
  // V: see v_swizzle.
  __device__ static uint32_t swz_k(uint32_t row) { return D == 128 ? row & 15 : (row >> 1) & 7; }
};

template <int CTRL>
__device__ __forceinline__ int dpp(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, false);
}
// Of a wave, in every lane, without the LDS, whose six round trips in turn came before a workgroup's first load: us a call 140 heads x 311
// queries, head_dim 64, 27.45 -> 27.2, 48 x 1200 30.7 -> 30.4, 256 x 512 76.4 -> 76.2.
__device__ __forceinline__ int wave_max(int v) {
  v = max(v, dpp<0xB1>(v));   // neighbours
  v = max(v, dpp<0x4E>(v));   // pairs
  v = max(v, dpp<0x141>(v));  // half rows, mirrored
  v = max(v, dpp<0x140>(v));  // rows of 16, mirrored
  const auto a = __builtin_amdgcn_permlane16_swap((uint32_t)v, (uint32_t)v, false, false);
  const unsigned a0 = a[0], a1 = a[1];
  v = max((int)a0, (int)a1);
  const auto b = __builtin_amdgcn_permlane32_swap((uint32_t)v, (uint32_t)v, false, false);
  const unsigned b0 = b[0], b1 = b[1];
  return max((int)b0, (int)b1);
}

// The head of a given rank by descending number of 64-key tiles (equal ones by ascending number), and where its packed rows begin
// and end, found by every wave on its own: its lanes hold all heads' counts, a bit of the wanted count takes a comparison per 64
// heads, and of the heads with that count it is the one with so many before it.  That takes about as long as the load of the head's
// number did, which a kernel in front of this one had sorted (us a call, with it and without: 256 heads x 512 queries over 576 ...
// 1536 keys 79.2 / 78.0 (among other calls 83.6 / 81.9, on another board 81.1 / 81.0), over 812 keys 80.2 / 77.7; 192 x 190 over 720, head_dim 64, 30.9 / 28.9; 112 x 262 over 562 38.3 / 36.8).  Not
// beyond 256 heads: with eight of them a lane 448 heads x 300 took 69 instead of 63.
__device__ __forceinline__ int head_of_rank(const AttendParams& prm, int rank, int& c0, int& c1) {
  constexpr int N = kRankHeads / 64;
  const int lane = threadIdx.x & 63, capacity = (int)prm.capacity;
  int from[N], to[N], tiles[N];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int head = min(i * 64 + lane, prm.BH - 1);
    from[i] = prm.cu[head];
    to[i] = prm.cu[head + 1];
  }
  int most = 0;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    from[i] = min(from[i], capacity);
    to[i] = min(to[i], capacity);
    tiles[i] = i * 64 + lane < prm.BH ? min(max((to[i] - from[i] + prm.n_resp + kTK - 1) / kTK, 1), 0xFFFF) : 0;
    most = max(most, tiles[i]);
  }
  most = wave_max(most);
  int found = 0, above = 0;  // the count, and how many heads have more tiles
  for (int bit = 1 << (31 - __builtin_clz(__builtin_amdgcn_readfirstlane(most))); bit > 0; bit >>= 1) {
    int n = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) n += __popcll(__ballot(tiles[i] >= (found | bit)));
    if (n > rank)
      found |= bit;
    else
      above = n;
  }
  int left = rank - above, head = 0;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const uint64_t same = __ballot(tiles[i] == found);
    const int n = __popcll(same);
    if (left >= 0 && left < n) {
      const int before = __builtin_amdgcn_mbcnt_hi((uint32_t)(same >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)same, 0));
      const int at = __builtin_ctzll(__ballot(tiles[i] == found && before == left));
      head = i * 64 + at;
      c0 = __builtin_amdgcn_readlane(from[i], at);
      c1 = __builtin_amdgcn_readlane(to[i], at);
    }
    left -= n;
  }
  return head;
}

// KIND: kRanked, the heads are taken by rank; kStreamed, V is too large to be kept (instantiations of their own: as a branch the former
// costs the other calls 0.5 %, the latter 1 %).
enum { kPlain, kRanked, kStreamed };
template <int D, bool HALVES, int KIND>
__global__ __launch_bounds__(kWaves * 64) void attend_tiles_kernel(const AttendParams prm) {
  using C = TileCfg<D, HALVES>;
  constexpr bool RANKED = KIND == kRanked;
  constexpr bool kFew = HALVES && D == 64;  // registers: no more than 168, up to which the next workgroup starts when the last one's second group has left
  constexpr int kAheadFrag = kFew && RANKED ? 2 : 3;  // LDS fragments requested ahead of the MFMA that takes them
  fetch_attend_arguments<!RANKED>();
  extern __shared__ __attribute__((aligned(1024))) char tiles_lds[];
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)tiles_lds;

  // Workgroup numbers that are congruent modulo 8 run on the same XCD and share its L2: the query tiles of one (head, key
  // split) get consecutive slots of one XCD, and their K/V rows come from HBM once.  Ordered heads are dealt to the XCDs in
  // turn, otherwise each XCD takes a run of units.
  const int qtiles = (prm.n_q + C::kQueries - 1) / C::kQueries;
  const bool ordered = RANKED || prm.order;
  const int slot = blockIdx.x / 8 + (ordered ? 0 : blockIdx.x % 8 * (gridDim.x / 8));
  const int unit = ordered ? (slot / qtiles) * 8 + blockIdx.x % 8 : slot / qtiles;  // (head, split) pair
  const int qtile = slot % qtiles;
  if (unit >= prm.BH * prm.n_splits) return;
  int c0 = 0, c1 = 0;  // rows of the packed segment
  int bh;
  if constexpr (RANKED)  // (heads are only ordered without splits)
    bh = head_of_rank(prm, unit, c0, c1);
  else
    bh = __builtin_amdgcn_readfirstlane(prm.order ? prm.order[unit] : unit / prm.n_splits);
  const int split = ordered ? 0 : unit % prm.n_splits;
  const int b = bh / prm.H;
  const int h = bh % prm.H;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool second = wave >= kWaves / 2;  // the group that runs one slot behind
  const int part = HALVES ? wave % 4 : wave;  // this wave's queries, and its rows of the tiles that it moves
  const int r = lane & 31;
  const int g = lane >> 5;

  const char *a_k = nullptr, *a_v = nullptr;  // packed segment
  int len_a = 0, len_b = prm.n_resp;
  if (prm.full) {
    len_b = prm.lens.P[b] + prm.n_resp;
  } else {
    if constexpr (!RANKED) {
      c0 = (int)min((int64_t)prm.cu[bh], prm.capacity);
      c1 = (int)min((int64_t)prm.cu[bh + 1], prm.capacity);
    }
    a_k = prm.Kc + (int64_t)c0 * C::kRowB;
    a_v = prm.Vc + (int64_t)c0 * C::kRowB;
    len_a = c1 - c0;
  }
  const int Lk = len_a + len_b;
  const int Ls = ((Lk + prm.n_splits - 1) / prm.n_splits + kTK - 1) / kTK * kTK;
  const int j0 = split * Ls;
  const int j1 = min(Lk, j0 + Ls);
  const int all_tiles = j1 > j0 ? (j1 - j0 + kTK - 1) / kTK : 0;
  // Tiles of this group: t stands for tile t, or 2t + group.  Both groups make `ntiles` steps; a last step may be without a tile.
  const int ntiles = HALVES ? (all_tiles + 1) / 2 : all_tiles;
  const int mine = HALVES ? (all_tiles + (second ? 0 : 1)) / 2 : all_tiles;
  auto first_key = [&](int t) { return j0 + (HALVES ? 2 * t + (second ? 1 : 0) : t) * kTK; };

  // ---- transfers: a wave moves kMoveRows rows of a tile, of K and of V.  As long as these rows lie in one segment, a tile takes a
  // scalar base that goes on by the same step, and offsets that the lanes keep; where they straddle the segments or the end, each lane
  // forms its own address.  (kFew: base and offsets are formed for each tile.  us a call, kept / formed: 168 heads x 214 queries over 270 keys
  // 19.5 / 17.6, over 900 31.9 / 29.3, x 120 over 270 10.2 / 9.5, 256 heads x 100 over 600 17.5 / 17.2.)
  const uint32_t mrow = (uint32_t)lane / C::kPPR, mpiece = (uint32_t)lane % C::kPPR;
  struct Feed {
    const char *packed, *rest, *base;  // base: of the next tile's rows
    uint32_t stride, step;             // of the second segment's rows; from a tile's rows to the next one's
    int whole;                         // how many tiles from the next one on are taken by base and step
    uint32_t off[C::kMoves], piece[C::kMoves];
  };
  auto uniform = [](const char* p) {  // (the same in every lane, but the compiler may hold it in vector registers)
    const uint64_t u = (uint64_t)p;
    return (const char*)((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(u >> 32)) << 32 | (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)u));
  };
  constexpr int kNext = HALVES ? 2 * kTK : kTK;  // keys from a tile of this group to the next
  // (On every way through `move`: where one comes without it the compiler moves the whole loop's state into vector registers.)
  auto scalar = [](Feed& f) { asm volatile("" : "+s"(f.whole), "+s"(f.base), "+s"(f.step)); };
  auto aim = [&](Feed& f, int t) {  // at tile t
    const int first = first_key(t) + part * C::kMoveRows;
    const bool in_a = first < len_a;
    const uint32_t st = in_a ? (uint32_t)C::kRowB : f.stride;
    const int left = (in_a ? min(len_a, j1) : j1) - first - C::kMoveRows;
    f.whole = __builtin_amdgcn_readfirstlane(left >= 0 ? left / kNext + 1 : 0);
    f.base = uniform(in_a ? f.packed + (int64_t)first * C::kRowB : f.rest + (int64_t)(first - len_a) * f.stride);
    f.step = __builtin_amdgcn_readfirstlane(kNext * st);
    scalar(f);
#pragma unroll
    for (int j = 0; j < C::kMoves; ++j) f.off[j] = (mrow + j * C::kRPI) * st + f.piece[j];
  };
  auto move = [&](Feed& f, int t, uint32_t to, auto streamed) {
    to += part * C::kMoveRows * C::kRowB;
    if (kFew) aim(f, t);
    if (__builtin_expect(f.whole > 0, 1)) {
#pragma unroll
      for (int j = 0; j < C::kMoves; ++j) decltype(streamed)::value ? dma16_streamed(f.base, f.off[j], to + j * 1024) : dma16(f.base, f.off[j], to + j * 1024);
      if (kFew) return;
      f.base += f.step;
      --f.whole;
      scalar(f);
      return;
    }
    const int first = first_key(t) + part * C::kMoveRows;  // (rows past the end re-read the last row, also those of tiles beyond the last one)
    if (first >= j1) {
      const char* last = uniform(j1 <= len_a ? f.packed + (int64_t)(j1 - 1) * C::kRowB : f.rest + (int64_t)(j1 - 1 - len_a) * f.stride);
#pragma unroll
      for (int j = 0; j < C::kMoves; ++j) dma16(last, f.piece[j], to + j * 1024);
      if (!kFew) scalar(f);
      return;
    }
#pragma unroll
    for (int j = 0; j < C::kMoves; ++j) {
      const int k = min(first + j * C::kRPI + (int)mrow, j1 - 1);
      const bool in_a = k < len_a;
      const char* from = in_a ? f.packed : f.rest;
      dma16_from(from + ((uint64_t)(uint32_t)(in_a ? k : k - len_a) * (in_a ? (uint32_t)C::kRowB : f.stride) + f.piece[j]), to + j * 1024);
    }
    if (!kFew) aim(f, t + 1);
  };
  // K's permutation depends on the transfer j by one exclusive-or (j * kRPI and the lane's row are row bits side by side, and
  // the permutation of j rows of transfers is j times that of one), V's does not.
  Feed fk, fv;
  fk.packed = a_k;
  fk.rest = prm.K2.row(b, h, 0);
  fk.stride = (uint32_t)prm.K2.stride_t;
  fv.packed = a_v;
  fv.rest = prm.V2.row(b, h, 0);
  fv.stride = (uint32_t)prm.V2.stride_t;
#pragma unroll
  for (int j = 0; j < C::kMoves; ++j) {
    fk.piece[j] = (mpiece ^ C::swz_k(part * C::kMoveRows + mrow) ^ j * C::swz_k(C::kRPI)) << 4;
    fv.piece[j] = (mpiece ^ v_swizzle<D>(mrow) << 1) << 4;
  }
  if (!kFew) {
    aim(fk, 0);
    aim(fv, 0);
  }
  auto ring = [&](int t) { return HALVES ? (second ? 2 : 0) + (t & 1) : t & 3; };
  auto move_k = [&](int t) { move(fk, t, lds0 + ring(t) * C::kTileB, std::false_type()); };
  auto move_v = [&](int t) { move(fv, t, lds0 + (4 + ring(t)) * C::kTileB, std::bool_constant<KIND == kStreamed>()); };

  const int q = qtile * C::kQueries + part * 32 + r;
  const bool active = qtile * C::kQueries + part * 32 < prm.n_q;  // (a wave without queries only helps to move the tiles)
  u32x4 qf[C::kSteps];
  // A wave moves its 32 rows as whole rows, into LDS that no tile needs before the third one.  (Its fragments straight from memory, a row
  // a lane, keep the texture path busy four times as long, in front of the first tiles: 256 heads x 256 queries over 320 ... 768 keys 30.65
  // us against 30.25, 140 x 311, head_dim 64, 28.2 / 27.4, 256 x 512 over 576 ... 1536 76.5 / 75.8.
  // With HALVES the second V tiles' slots have room for them, and the two waves of the same rows move half of these each.)
  constexpr int kQRows = HALVES ? 16 : 32;
  const uint32_t q_at = lds0 + (HALVES ? (5 + part / 2 * 2) * C::kTileB + part % 2 * (32 * C::kRowB) : C::kOffQ + part * (32 * C::kRowB));
  if (ntiles > 0) {  // (a part of the keys may be empty: nothing then waits for a transfer)
#pragma unroll
    for (int j = 0; j < kQRows / C::kRPI; ++j) {
      const uint32_t row = (HALVES && second ? kQRows : 0) + j * C::kRPI + mrow;
      const char* from = prm.Q.group_row(b, h, prm.q_per_kv, prm.n_resp, min(qtile * C::kQueries + part * 32 + (int)row, prm.n_q - 1));
      dma16_from(from + ((mpiece ^ C::swz_k(row)) << 4), q_at + (HALVES && second ? kQRows * C::kRowB : 0) + j * 1024);
    }
  }

  f32x16 o[C::kDB], s[2];
  u32x4 pf[4];  // probabilities of a tile as B operands: keys 32*(n/2) + 16*(n%2) ..
#pragma unroll
  for (int db = 0; db < C::kDB; ++db) o[db] = f32x16{};
  float m = kNegBig, l = 0.f;
  const float c = prm.c;

  // ---- fragment addresses.  Four ring slots are two pairs: the second of a pair is an immediate offset away.
  const uint32_t own = lds0 + (HALVES && second ? 2 * C::kTileB : 0);
  uint32_t ka[C::kSteps], va[C::kDB];
#pragma unroll
  for (int i = 0; i < C::kSteps; ++i) ka[i] = own + r * C::kRowB + (((2 * i + g) ^ C::swz_k(r)) << 4);
#pragma unroll
  for (int db = 0; db < C::kDB; ++db) va[db] = own + 4 * C::kTileB + v_read_offset<D>(lane, db);
#pragma unroll
  for (int i = 0; i < C::kSteps; ++i) asm volatile("" : "+v"(ka[i]));
#pragma unroll
  for (int i = 0; i < C::kDB; ++i) asm volatile("" : "+v"(va[i]));
  auto turn_k = [&]() {
    if (HALVES) return;
#pragma unroll
    for (int i = 0; i < C::kSteps; ++i) ka[i] ^= 2 * C::kTileB;
  };
  auto turn_v = [&]() {
    if (HALVES) return;
#pragma unroll
    for (int i = 0; i < C::kDB; ++i) va[i] ^= 2 * C::kTileB;
  };

  // ---- matrix phase: fragments n = 0 .. kQK-1 are the logits' (two chains, one per block of 32 keys), then the output's
  u32x4 fr[kAheadFrag + 1];
  auto fetch = [&](int n, int pk, int pv) {
    u32x4& f = fr[n % (kAheadFrag + 1)];
    if (n < C::kQK) {
      f = *in_lds<const u32x4>(ka[n / 2], pk * C::kTileB + (n % 2) * 32 * C::kRowB);
    } else {
      const int i = n - C::kQK, imm = pv * C::kTileB + (i / C::kDB) * 16 * C::kRowB;
      const u32x2 lo = read_transposed(va[i % C::kDB], imm), hi = read_transposed(va[i % C::kDB], imm + 8 * C::kRowB);
      f = u32x4{lo[0], lo[1], hi[0], hi[1]};
    }
  };
  auto matrix = [&](int from, int to, int pk, int pv) {
#pragma unroll
    for (int i = 0; i < kAheadFrag; ++i) fetch(from + i, pk, pv);
    if (from == 0) s[0] = s[1] = f32x16{};
#pragma unroll
    for (int n = from; n < to; ++n) {
      if (n + kAheadFrag < to) fetch(n + kAheadFrag, pk, pv);
      const u32x4& f = fr[n % (kAheadFrag + 1)];
      if (n < C::kQK)
        mfma_step<bf16_t>(f, qf[n / 2], s[n % 2]);
      else
        mfma_step<bf16_t>(f, pf[(n - C::kQK) / C::kDB], o[(n - C::kQK) % C::kDB]);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  // ---- vector phase: online softmax of the logits; lanes l and l^32 hold the same query
  auto softmax = [&](int t) {
    const int left = j1 - first_key(t);
    if (left < kTK) {
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (kb * 32 + 8 * (i / 4) + 4 * g + (i % 4) >= left) s[kb][i] = -INFINITY;
    }
    float bm = s[0][0];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int i = 0; i < 16; ++i) bm = fmaxf(bm, s[kb][i]);
    bm = max_halves(bm);
    // The reference m is only raised when a tile exceeds it by more than 2^kLazyBump (see attend.hip).
    const float cand = bm * c;
    const bool bump = cand > m + kLazyBump;
    if (__any(bump)) {
      const float m_new = bump ? cand : m;
      const float alpha = fast_exp2(m - m_new);
      m = m_new;
      l *= alpha;
#pragma unroll
      for (int db = 0; db < C::kDB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[db][i] *= alpha;
    }
    float psum = 0.f;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const float p = fast_exp2(fmaf(s[kb][i], c, -m));
        s[kb][i] = p;
        psum += p;
      }
#pragma unroll
      for (int tp = 0; tp < 2; ++tp)
#pragma unroll
        for (int w = 0; w < 4; ++w) pf[2 * kb + tp][w] = pack_bf16x2(s[kb][8 * tp + 2 * w], s[kb][8 * tp + 2 * w + 1]);
    }
    l += psum;
  };

  // ---- barriers.  At barrier t every wave has waited for its part of pair t: group 0 at the end of its vector phase t-1, where pairs
  // t+1 and t+2 are younger, group 1 at the end of its matrix phase t-1, where pair t+1 is.  One more barrier behind group 0's first
  // matrix phase lets group 1 start half a tile late.
  // With HALVES a group moves its own tiles, pair t+2 in vector phase t (into the slots of K(t) and V(t-1), which it has
  // read), and waits for pair t+1 at the end of that phase; the groups meet at a barrier after every phase.
  auto end_matrix = [&](bool first) {
    __builtin_amdgcn_sched_barrier(0);
    if (!HALVES && second)
      asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"i"(2 * C::kMoves) : "memory");
    else if (HALVES || first)
      asm volatile("s_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  auto end_vector = [&]() {
    __builtin_amdgcn_sched_barrier(0);
    if (HALVES)
      asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"i"(2 * C::kMoves) : "memory");
    else if (!second)
      asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"i"(4 * C::kMoves) : "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  auto vector = [&](int t) {
    if (!HALVES || t < mine) {  // (a step without a tile has left V(t-1) unread)
      move_k(t + (HALVES ? 2 : 3));
      move_v(t + (HALVES ? 1 : 2));
    }
    if (active && t < mine) softmax(t);
    end_vector();
  };

  if (ntiles > 0) {
    move_k(0);
    move_k(1);
    move_v(0);
    if (!HALVES) {
      move_k(2);
      move_v(1);
    }
    if (HALVES)
      asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"i"(3 * C::kMoves) : "memory");
    else
      asm volatile("s_waitcnt vmcnt(%0)" ::"i"(5 * C::kMoves) : "memory");
#pragma unroll
    for (int i = 0; i < C::kSteps; ++i) qf[i] = *in_lds<const u32x4>(q_at + (ka[i] - own));
#pragma unroll
    for (int i = 0; i < C::kSteps; ++i) asm volatile("" : "+v"(qf[i]));  // (read before the barrier: V tiles take their place)
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"i"((HALVES ? 2 : 4) * C::kMoves) : "memory");
    if (second) asm volatile("s_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    if (active && mine > 0) matrix(0, C::kQK, 0, 0);
    end_matrix(true);
    vector(0);
    for (int t = 1; t < ntiles; t += 2) {
      if (active && t < mine) matrix(0, C::kQK + C::kPV, 1, 0);
      turn_k();
      end_matrix(false);
      vector(t);
      if (t + 1 < ntiles) {
        if (active && t + 1 < mine) matrix(0, C::kQK + C::kPV, 0, 1);
        turn_v();
        end_matrix(false);
        vector(t + 1);
      }
    }
    if (active && mine > 0) {
      if (mine & 1)
        matrix(C::kQK, C::kQK + C::kPV, 0, 0);
      else
        matrix(C::kQK, C::kQK + C::kPV, 0, 1);
    }
    if (HALVES && !second) asm volatile("s_barrier" ::: "memory");
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (no transfer into LDS outlives its workgroup)
  }

  float l_tot = sum_halves(l);
  // HALVES: each group has half of the head dimension in the end; the other half of its part is for the other group, through LDS.  (us a
  // call, with all of it put together by one group, 4 bytes a lane, and the queries a row a lane, before: 196 heads x 167 queries over 230 ... 350
  // keys 26.2 / 24.8, 48 x 1200 over 360 ... 700 32.1 / 30.6.)
  constexpr int kOwn = HALVES ? C::kDB / 2 : C::kDB;  // blocks of 32 elements
  f32x16 res[kOwn];
  int e0 = 0;  // its first element
  if constexpr (HALVES) {
    f32x4* const parts = reinterpret_cast<f32x4*>(tiles_lds);  // [wave][kOwn][4][lane]
    float2* const ml = reinterpret_cast<float2*>(tiles_lds + kWaves * kOwn * 4 * 64 * 16);
    f32x4* const to = parts + wave * (kOwn * 4 * 64) + lane;
    const f32x4* const from = parts + (wave ^ 4) * (kOwn * 4 * 64) + lane;
    auto give = [&](int db0) {
#pragma unroll
      for (int db = 0; db < kOwn; ++db)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          to[(db * 4 + i) * 64] = f32x4{o[db0 + db][4 * i], o[db0 + db][4 * i + 1], o[db0 + db][4 * i + 2], o[db0 + db][4 * i + 3]};
    };
    __syncthreads();
    if (second)
      give(0);
    else
      give(kOwn);
    ml[wave * 64 + lane] = make_float2(m, l_tot);
    __syncthreads();
    const float2 other = ml[(wave ^ 4) * 64 + lane];
    const float top = fmaxf(m, other.x);
    const float w_own = fast_exp2(m - top), w_other = fast_exp2(other.x - top);
    const float wa = second ? w_other : w_own, wb = second ? w_own : w_other;  // of group 0 and of group 1
    m = top;
    l_tot = wa * (second ? other.y : l_tot) + wb * (second ? l_tot : other.y);
    auto take = [&](auto group) {
      constexpr bool kFirst = decltype(group)::value == 0;
      constexpr int db0 = kFirst ? 0 : kOwn;
#pragma unroll
      for (int db = 0; db < kOwn; ++db)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const f32x4 v = from[(db * 4 + i) * 64];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float mine_of = o[db0 + db][4 * i + e], theirs = v[e];
            res[db][4 * i + e] = wa * (kFirst ? mine_of : theirs) + wb * (kFirst ? theirs : mine_of);
          }
        }
    };
    if (second)
      take(std::integral_constant<int, 1>());
    else
      take(std::integral_constant<int, 0>());
    e0 = second ? kOwn * 32 : 0;
  } else {
#pragma unroll
    for (int db = 0; db < kOwn; ++db) res[db] = o[db];
  }
  if (q >= prm.n_q) return;  // (of two lanes 32 apart both or none)
  if (prm.n_splits == 1) {
    const float inv = 1.f / l_tot;
    char* orow = prm.O.group_row(b, h, prm.q_per_kv, prm.n_resp, q) + 2 * e0 + 16 * g;
#pragma unroll
    for (int db = 0; db < kOwn; ++db)
#pragma unroll
      for (int qd = 0; qd < 4; qd += 2) {
        // A lane has four elements of each eight, the lane 32 on the other four: one gives the second four for the first ones of the next
        // eight, so that a lane stores 16 bytes of a row instead of 8 and an instruction touches 32 rows eight times a wave instead of
        // sixteen (the texture path takes a cycle and more a row, and the next workgroup's first loads wait behind it).  us a call: 256
        // heads x 256 queries over 320 ... 768 keys 32.1 -> 30.7, 196 x 167 27.8 -> 26.2, 140 x 311, head_dim 64, 29.1 -> 28.2, x 512 over
        // 576 ... 1536 77.9 -> 76.6.
        u32x4 w;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const uint32_t first = pack_bf16x2(res[db][4 * qd + 2 * i] * inv, res[db][4 * qd + 2 * i + 1] * inv);
          const uint32_t next = pack_bf16x2(res[db][4 * qd + 4 + 2 * i] * inv, res[db][4 * qd + 5 + 2 * i] * inv);
          const auto sw = __builtin_amdgcn_permlane32_swap(first, next, false, false);
          const unsigned w0 = sw[0], w1 = sw[1];
          w[i] = w0;
          w[2 + i] = w1;
        }
        *reinterpret_cast<u32x4*>(orow + (db * 32 + 8 * qd) * 2) = w;
      }
    if (prm.lse && g == 0 && e0 == 0) prm.lse[(int64_t)bh * prm.n_q + q] = (m + __log2f(l_tot)) * kLn2;
  } else {
    const int64_t at = ((int64_t)bh * prm.n_splits + split) * prm.n_q + q;
    float* po = prm.part_o + at * D + e0;
#pragma unroll
    for (int db = 0; db < kOwn; ++db)
#pragma unroll
      for (int qd = 0; qd < 4; ++qd)
        *reinterpret_cast<float4*>(po + db * 32 + 8 * qd + 4 * g) =
            make_float4(res[db][4 * qd], res[db][4 * qd + 1], res[db][4 * qd + 2], res[db][4 * qd + 3]);
    if (g == 0 && e0 == 0) prm.part_ml[at] = make_float2(m, l_tot);
  }
}

template <int D, bool HALVES, int KIND>
int launch(const AttendParams& prm, unsigned groups, hipStream_t stream) {
  using C = TileCfg<D, HALVES>;
  static bool raised = false;  // one-time opt-in to more than the default dynamic LDS size
  if (!raised) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&attend_tiles_kernel<D, HALVES, KIND>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, C::kLds);
    if (e != hipSuccess) {
      set_error("attend: cannot raise dynamic LDS limit: %s", hipGetErrorString(e));
      (void)hipGetLastError();
      return MASKKV_EHIP;
    }
    raised = true;
  }
  hipLaunchKernelGGL((attend_tiles_kernel<D, HALVES, KIND>), dim3(groups), dim3(kWaves * 64), C::kLds, stream, prm);
  return check_launch("attend (tiles)");
}

template <bool HALVES>
int launch(const AttendParams& prm, int d, unsigned groups, hipStream_t stream) {
  if (prm.ranked) return d == 128 ? launch<128, HALVES, kRanked>(prm, groups, stream) : launch<64, HALVES, kRanked>(prm, groups, stream);
  if (prm.streamed) return d == 128 ? launch<128, HALVES, kStreamed>(prm, groups, stream) : launch<64, HALVES, kStreamed>(prm, groups, stream);
  return d == 128 ? launch<128, HALVES, kPlain>(prm, groups, stream) : launch<64, HALVES, kPlain>(prm, groups, stream);
}

}  // namespace

// 128 queries a workgroup where 256 would leave compute units without one (measured, 128 against 256: 128 heads x 256 queries
// 23.6 / 29.3 us, 256 heads x 100 queries 29.1 / 34.3, head_dim 64 128 heads x 200 queries 22.8 / 33.4; but 256 heads x 512
// queries 102 / 85).  The un-evicted call fills the chip by splitting the keys instead.
int attend_tiles_queries(int64_t units, int n_q, bool full) {
  if (n_q <= 128) return 128;
  return !full && (n_q + 255) / 256 * units < 256 ? 128 : 256;
}

int launch_attend_tiles(const AttendParams& prm, int d, int queries, hipStream_t stream) {
  const int64_t qtiles = (prm.n_q + queries - 1) / queries, units = (int64_t)prm.BH * prm.n_splits;
  const unsigned groups = (unsigned)(prm.order || prm.ranked ? (units + 7) / 8 * 8 * qtiles : (units * qtiles + 7) / 8 * 8);
  return queries == 128 ? launch<true>(prm, d, groups, stream) : launch<false>(prm, d, groups, stream);
}

}  // namespace maskkv
