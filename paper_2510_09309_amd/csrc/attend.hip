// Bidirectional attention of the response span over [kept prompt KV ; response KV]
// (MaskKV Section 3.1 layer forward equation; appendix: AttnOut_m = sum_j alpha_mj V_j), and the
// same attention over the un-evicted sequence.
//
// Flash-style single pass with an online softmax.  The logits are formed transposed (keys on the MFMA row axis, queries on
// the column axis), so a lane owns one query: its running max / sum stay in the lane and the probabilities it holds are
// already laid out as the B operand of O^T = V^T P^T.  The key axis is the concatenation of two segments (packed cache rows,
// then a strided view; the narrow bf16 kernel takes the view first); long key axes are split across workgroups and merged by a
// second small kernel.
//
// Here: the tiled kernel for fp32 (8 waves = 256 queries of one (b, h) sharing every staged K/V tile, V written to LDS
// transposed so that the A operand of the second product is read with 16-byte LDS loads), the narrow kernels for small
// launches, the merge and the rules that choose.  attend_tiles.hip: the tiled kernel for bf16.
#include "attend.hpp"
#include "lds.hpp"

namespace maskkv {

namespace {

constexpr int kUnits = 256;  // compute units

template <int D>
struct AttCfg {
  static constexpr int kEB = 4;  // bytes per element
  static constexpr int kRowB = D * kEB;
  static constexpr int kRowP = kRowB + 16;
  static constexpr int kSteps = kRowB / 32;
  static constexpr int kTK = (kRowB <= 256) ? 64 : 32;
  static constexpr int kNKB = kTK / 32;
  static constexpr int kPiecesPerRow = kRowB / 16;
  static constexpr int kWaves = 8;  // waves (32 queries each) that share a K/V tile
  static constexpr int kThreads = kWaves * 64;
  static constexpr int kQPerBlock = kWaves * 32;
  static constexpr int kPieces = kTK * kRowB / 16 / kThreads;
  static constexpr int kSV = kTK + 4;  // elements per transposed-V row (padding keeps LDS reads conflict-free)
  static constexpr int kDB = D / 32;
  static constexpr int kKtBytes = kTK * kRowP;
  static constexpr int kVtBytes = D * kSV * kEB;
  static constexpr int kLds = 2 * (kKtBytes + kVtBytes);  // K and V^T tiles, double-buffered
};

template <int D>
__device__ __forceinline__ void load_kv(const AttendParams& prm, const KeySpace& ks, int b, int h, int key0, int klast,
                                        u32x4 (&kr)[AttCfg<D>::kPieces], u32x4 (&vr)[AttCfg<D>::kPieces]) {
  using C = AttCfg<D>;
#pragma unroll
  for (int i = 0; i < C::kPieces; ++i) {
    const int p = threadIdx.x + i * C::kThreads;
    {
      const int row = p / C::kPiecesPerRow, col = p % C::kPiecesPerRow;
      const int j = min(key0 + row, klast);
      const char* src = j < ks.len_a ? ks.a_k + (int64_t)j * C::kRowB : prm.K2.row(b, h, j - ks.len_a);
      kr[i] = *reinterpret_cast<const u32x4*>(src + col * 16);
    }
    {
      const int row = p / C::kPiecesPerRow, col = p % C::kPiecesPerRow;
      const int j = min(key0 + row, klast);
      const char* src = j < ks.len_a ? ks.a_v + (int64_t)j * C::kRowB : prm.V2.row(b, h, j - ks.len_a);
      vr[i] = *reinterpret_cast<const u32x4*>(src + col * 16);
    }
  }
}

template <int D>
__device__ __forceinline__ void store_kv(char* kt, char* vt, const u32x4 (&kr)[AttCfg<D>::kPieces],
                                         const u32x4 (&vr)[AttCfg<D>::kPieces]) {
  using C = AttCfg<D>;
#pragma unroll
  for (int i = 0; i < C::kPieces; ++i) {
    const int p = threadIdx.x + i * C::kThreads;
    const int row = p / C::kPiecesPerRow, col = p % C::kPiecesPerRow;
    *reinterpret_cast<u32x4*>(kt + row * C::kRowP + col * 16) = kr[i];
  }
  uint32_t* vt32 = reinterpret_cast<uint32_t*>(vt);
#pragma unroll
  for (int i = 0; i < C::kPieces; ++i) {
    const int p = threadIdx.x + i * C::kThreads;
    const int row = p / C::kPiecesPerRow, col = p % C::kPiecesPerRow;
#pragma unroll
    for (int w = 0; w < 4; ++w) vt32[(col * 4 + w) * C::kSV + row] = vr[i][w];
  }
}

template <int D>
__global__ __launch_bounds__((AttCfg<D>::kThreads)) void attend_kernel(const AttendParams prm) {
  using C = AttCfg<D>;
  extern __shared__ __attribute__((aligned(16))) char att_lds[];  // two buffers of (K tile, V^T tile)

  // Workgroup numbers that are congruent modulo 8 run on the same XCD and share its L2.  The query tiles of
  // one (head, key split) read the same K/V rows, so they are given consecutive slots of one XCD: the rows
  // then come from HBM once instead of once per query tile.
  const int qtiles = (prm.n_q + C::kQPerBlock - 1) / C::kQPerBlock;
  const int slot = blockIdx.x / 8;
  const int unit = (slot / qtiles) * 8 + blockIdx.x % 8;  // (head, split) pair
  const int qtile = slot % qtiles;
  if (unit >= prm.BH * prm.n_splits) return;
  const int bh = prm.order ? prm.order[unit] : unit / prm.n_splits;  // (an order is only given without splits)
  const int split = prm.order ? 0 : unit % prm.n_splits;
  const int b = bh / prm.H;
  const int h = bh % prm.H;
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int r = lane & 31;
  const int g = lane >> 5;

  KeySpace ks;
  if (prm.full) {
    ks.a_k = ks.a_v = nullptr;
    ks.len_a = 0;
    ks.len_b = prm.lens.P[b] + prm.n_resp;
  } else {
    const int64_t c0 = min((int64_t)prm.cu[bh], prm.capacity);
    const int64_t c1 = min((int64_t)prm.cu[bh + 1], prm.capacity);
    ks.a_k = prm.Kc + c0 * C::kRowB;
    ks.a_v = prm.Vc + c0 * C::kRowB;
    ks.len_a = (int)(c1 - c0);
    ks.len_b = prm.n_resp;
  }
  const int Lk = ks.len_a + ks.len_b;
  const int Ls = ((Lk + prm.n_splits - 1) / prm.n_splits + C::kTK - 1) / C::kTK * C::kTK;
  const int j0 = split * Ls;
  const int j1 = min(Lk, j0 + Ls);
  const int ntiles = j1 > j0 ? (j1 - j0 + C::kTK - 1) / C::kTK : 0;

  const int q = qtile * C::kQPerBlock + wave * 32 + r;
  u32x4 qf[C::kSteps];
#pragma unroll
  for (int s = 0; s < C::kSteps; ++s) {
    if (q < prm.n_q)
      qf[s] = *reinterpret_cast<const u32x4*>(prm.Q.group_row(b, h, prm.q_per_kv, prm.n_resp, q) + s * 32 + g * 16);
    else
      qf[s] = u32x4{0u, 0u, 0u, 0u};
  }

  f32x16 o[C::kDB];
#pragma unroll
  for (int db = 0; db < C::kDB; ++db) o[db] = f32x16{};
  float m = kNegBig, l = 0.f;
  const float c = prm.c;

  // Two tiles are kept in flight in two register sets (a key axis of a few hundred rows is a short serial
  // chain of tiles, so the memory latency of each request has to hide behind two tiles of arithmetic).
  u32x4 kra[C::kPieces], vra[C::kPieces], krb[C::kPieces], vrb[C::kPieces];
  // Tile t is computed from LDS buffer t&1 while tile t+1 is written to the other one: one barrier per tile.
  if (ntiles > 0) load_kv<D>(prm, ks, b, h, j0, j1 - 1, kra, vra);
  if (ntiles > 1) load_kv<D>(prm, ks, b, h, j0 + C::kTK, j1 - 1, krb, vrb);
  if (ntiles > 0) {
    store_kv<D>(att_lds, att_lds + C::kKtBytes, kra, vra);
    if (ntiles > 2) load_kv<D>(prm, ks, b, h, j0 + 2 * C::kTK, j1 - 1, kra, vra);
  }
  __syncthreads();

  // `kr`, `vr` hold tile t+1 on entry (if there is one) and are refilled with tile t+3.
  auto tile_step = [&](int t, u32x4 (&kr)[C::kPieces], u32x4 (&vr)[C::kPieces]) {
    const int key0 = j0 + t * C::kTK;
    const char* kt = att_lds + (t & 1) * (C::kKtBytes + C::kVtBytes);
    const char* vt = kt + C::kKtBytes;
    if (t + 1 < ntiles) {  // the other buffer's readers (tile t-1) passed the barrier that ended the previous step
      char* nk = att_lds + ((t + 1) & 1) * (C::kKtBytes + C::kVtBytes);
      store_kv<D>(nk, nk + C::kKtBytes, kr, vr);
      if (t + 3 < ntiles) load_kv<D>(prm, ks, b, h, key0 + 3 * C::kTK, j1 - 1, kr, vr);
    }

    // S^T = K Q^T for this tile
    f32x16 s[C::kNKB];
#pragma unroll
    for (int kb = 0; kb < C::kNKB; ++kb) {
      s[kb] = f32x16{};
#pragma unroll
      for (int st = 0; st < C::kSteps; ++st) {
        const u32x4 kf = *reinterpret_cast<const u32x4*>(kt + (kb * 32 + r) * C::kRowP + st * 32 + g * 16);
        mfma_step<float>(kf, qf[st], s[kb]);
      }
      const int nvalid = j1 - (key0 + kb * 32);
      if (nvalid < 32) {
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (8 * (i / 4) + 4 * g + (i % 4) >= nvalid) s[kb][i] = -INFINITY;
      }
    }
    // online softmax; lanes l and l^32 hold the same query
    float bm = s[0][0];
#pragma unroll
    for (int kb = 0; kb < C::kNKB; ++kb)
#pragma unroll
      for (int i = 0; i < 16; ++i) bm = fmaxf(bm, s[kb][i]);
    bm = max_halves(bm);
    // The reference m is only raised when a tile exceeds it by more than 2^kLazyBump: probabilities then stay
    // below 2^kLazyBump (harmless in fp32 sums and as bf16 operands, whose exponent range is fp32's), and the
    // accumulators are rescaled on few tiles only.
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
    for (int kb = 0; kb < C::kNKB; ++kb)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const float p = fast_exp2(fmaf(s[kb][i], c, -m));
        s[kb][i] = p;
        psum += p;
      }
    l += psum;

    // O^T += V^T P^T
#pragma unroll
    for (int kb = 0; kb < C::kNKB; ++kb)
#pragma unroll
      for (int qd = 0; qd < 4; ++qd) {
        u32x4 pf;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const float pv = s[kb][4 * qd + w];
          pf[w] = as_u32(pv);
        }
#pragma unroll
        for (int db = 0; db < C::kDB; ++db) {
          const u32x4 vf = *reinterpret_cast<const u32x4*>(vt + ((db * 32 + r) * C::kSV + kb * 32 + 8 * qd + 4 * g) * 4);
          mfma_step<float>(vf, pf, o[db]);
        }
      }
    __syncthreads();  // tile t+1 is visible; every wave is done with tile t
  };
  for (int t = 0; t < ntiles; t += 2) {
    tile_step(t, krb, vrb);
    if (t + 1 < ntiles) tile_step(t + 1, kra, vra);
  }

  const float l_tot = sum_halves(l);
  if (q >= prm.n_q) return;
  if (prm.n_splits == 1) {
    const float inv = 1.f / l_tot;
    char* orow = prm.O.group_row(b, h, prm.q_per_kv, prm.n_resp, q);
#pragma unroll
    for (int db = 0; db < C::kDB; ++db)
#pragma unroll
      for (int qd = 0; qd < 4; ++qd) {
        const int e = db * 32 + 8 * qd + 4 * g;
        const float v0 = o[db][4 * qd] * inv, v1 = o[db][4 * qd + 1] * inv;
        const float v2 = o[db][4 * qd + 2] * inv, v3 = o[db][4 * qd + 3] * inv;
        *reinterpret_cast<float4*>(orow + e * 4) = make_float4(v0, v1, v2, v3);
      }
    if (prm.lse && g == 0) prm.lse[(int64_t)bh * prm.n_q + q] = (m + __log2f(l_tot)) * kLn2;
  } else {
    const int64_t slot = ((int64_t)bh * prm.n_splits + split) * prm.n_q + q;
    float* po = prm.part_o + slot * D;
#pragma unroll
    for (int db = 0; db < C::kDB; ++db)
#pragma unroll
      for (int qd = 0; qd < 4; ++qd) {
        const int e = db * 32 + 8 * qd + 4 * g;
        *reinterpret_cast<float4*>(po + e) =
            make_float4(o[db][4 * qd], o[db][4 * qd + 1], o[db][4 * qd + 2], o[db][4 * qd + 3]);
      }
    if (g == 0) prm.part_ml[slot] = make_float2(m, l_tot);
  }
}

// ---------------------------------------------------------------------------------------------
// Narrow launches (few heads x query tiles): a tiled kernel would occupy a fraction of the compute units with one long serial
// chain of tiles each.  Here a workgroup serves 32 queries and its waves split the key axis: wave w of n takes the 32-key
// blocks w, w + n, ... on its own, no workgroup barrier in the loop, and the partial (O, m, l) are merged through LDS at the
// end.  Every XCD (workgroup numbers that are congruent modulo 8) takes one run of (head, query tile) pairs, so that a head's K/V
// rows are fetched into one or two L2s and four heads still reach all eight XCDs (4 heads x 1792 queries: 23.7 us with a head on
// one XCD, 12.6 spread).
//
// fp32, 32 queries: four waves, K fragments from global memory into registers, V through a wave-private transposed LDS tile, two blocks in flight.
constexpr int kNarrowVS = 36;      // elements per transposed-V row: 32 keys + padding
constexpr int kNarrowShift = 16;   // bytes by which every group of 32 rows is shifted further

template <int D>
struct NarrowCfg {
  static constexpr int kWaves = 4;  // that split the key axis
  static constexpr int kEB = 4;
  static constexpr int kThreads = 64 * kWaves;
  static constexpr int kRowB = D * kEB;
  static constexpr int kSteps = kRowB / 32;
  static constexpr int kPPR = kRowB / 16;        // 16-byte pieces per row
  static constexpr int kVP = 32 * kPPR / 64;     // V pieces per lane per block
  static constexpr int kDB = D / 32;
  static constexpr int kSets = kRowB <= 256 ? 2 : 1;  // blocks a wave keeps in flight (512-byte rows: registers for one)
  static constexpr int kVtBytes = D * kNarrowVS * kEB + (D / 32) * kNarrowShift;  // per wave
  static constexpr int kMergeBytes = kWaves * kDB * 16 * 64 * 4;                   // partial O of the waves
  static constexpr int kLds = (kMergeBytes > kWaves * kVtBytes ? kMergeBytes : kWaves * kVtBytes) + kWaves * 32 * 8;
};

template <int D>
__global__ __launch_bounds__(NarrowCfg<D>::kThreads) void attend_narrow_kernel(const AttendParams prm) {
  fetch_attend_arguments<true>();
  using C = NarrowCfg<D>;
  constexpr int NW = C::kWaves;
  extern __shared__ __attribute__((aligned(16))) char smem[];

  const int nqt = (prm.n_q + 31) / 32;
  // eight runs of consecutive (head, query tile) pairs, one per XCD
  const int pair = (blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8;
  const int bh = pair / nqt;
  const int qt = pair % nqt;
  if (bh >= prm.BH) return;
  const int b = bh / prm.H;
  const int h = bh % prm.H;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane & 31;
  const int g = lane >> 5;

  int64_t c0 = 0, c1 = 0;
  if (!prm.full) {
    c0 = min((int64_t)prm.cu[bh], prm.capacity);
    c1 = min((int64_t)prm.cu[bh + 1], prm.capacity);
  }
  const char* a_k = prm.Kc + c0 * C::kRowB;
  const char* a_v = prm.Vc + c0 * C::kRowB;
  const int len_a = (int)(c1 - c0);
  const int Lk = len_a + prm.n_resp + (prm.full ? prm.lens.P[b] : 0);
  const int nblk = (Lk + 31) / 32;

  auto key_row = [&](const char* packed, const View& rest, int j) -> const char* {
    return j < len_a ? packed + (int64_t)j * C::kRowB : rest.row(b, h, j - len_a);
  };
  // Ask for block blk: K in MFMA fragment layout (lane = key row), V as row pieces for the transposition.  Rows past the end of the
  // key axis re-read its last row and are masked.
  auto request = [&](int blk, u32x4 (&kf)[C::kSteps], u32x4 (&vr)[C::kVP]) {
#pragma unroll
    for (int i = 0; i < C::kVP; ++i) {
      const int p = lane + i * 64;
      vr[i] = *reinterpret_cast<const u32x4*>(key_row(a_v, prm.V2, min(blk * 32 + p / C::kPPR, Lk - 1)) + p % C::kPPR * 16);
    }
    const char* krow = key_row(a_k, prm.K2, min(blk * 32 + r, Lk - 1)) + g * 16;
#pragma unroll
    for (int s = 0; s < C::kSteps; ++s) kf[s] = *reinterpret_cast<const u32x4*>(krow + s * 32);
  };

  // the first blocks of this wave are asked for before anything else: their latency covers the query loads
  u32x4 kfa[C::kSteps], vra[C::kVP], kfb[C::kSteps], vrb[C::kVP];
  if (wave < nblk) request(wave, kfa, vra);
  if (C::kSets == 2 && wave + NW < nblk) request(wave + NW, kfb, vrb);

  const int q = qt * 32 + r;
  u32x4 qf[C::kSteps];
  {
    const char* qrow = prm.Q.group_row(b, h, prm.q_per_kv, prm.n_resp, min(q, prm.n_q - 1));
#pragma unroll
    for (int s = 0; s < C::kSteps; ++s) qf[s] = *reinterpret_cast<const u32x4*>(qrow + s * 32 + g * 16);
  }
  f32x16 o[C::kDB];
#pragma unroll
  for (int db = 0; db < C::kDB; ++db) o[db] = f32x16{};
  float m = kNegBig, l = 0.f;
  const float c = prm.c;
  uint32_t* vt32 = reinterpret_cast<uint32_t*>(smem + wave * C::kVtBytes);

  auto step = [&](int blk, u32x4 (&kf)[C::kSteps], u32x4 (&vr)[C::kVP]) {
    // V^T of the block into this wave's LDS tile.  The tile is private to the wave; the fences order this block's
    // stores after the previous block's fragment loads and before this block's.
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int i = 0; i < C::kVP; ++i) {
      const int p = lane + i * 64, row = p / C::kPPR, col = p % C::kPPR;
#pragma unroll
      for (int w = 0; w < 4; ++w) vt32[(col * 4 + w) * kNarrowVS + (col / 8) * (kNarrowShift / 4) + row] = vr[i][w];
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    // S^T = K Q^T: keys on rows, queries on columns
    f32x16 s = f32x16{};
#pragma unroll
    for (int st = 0; st < C::kSteps; ++st) mfma_step<float>(kf[st], qf[st], s);
    if (blk + C::kSets * NW < nblk) request(blk + C::kSets * NW, kf, vr);
    const int nvalid = Lk - blk * 32;
    if (nvalid < 32) {
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (8 * (i / 4) + 4 * g + (i % 4) >= nvalid) s[i] = -INFINITY;
    }
    // online softmax; lanes l and l^32 hold the same query
    float bm = s[0];
#pragma unroll
    for (int i = 1; i < 16; ++i) bm = fmaxf(bm, s[i]);
    bm = max_halves(bm);
    const float cand = bm * c;
    const bool bump = cand > m + kLazyBump;  // the reference is raised lazily, as in the tiled kernel
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
    for (int i = 0; i < 16; ++i) {
      const float pv = fast_exp2(fmaf(s[i], c, -m));
      s[i] = pv;
      psum += pv;
    }
    l += psum;
    // O^T += V^T P^T
    const char* vt = reinterpret_cast<const char*>(vt32);
#pragma unroll
    for (int qd = 0; qd < 4; ++qd) {
      const u32x4 pf = {as_u32(s[4 * qd]), as_u32(s[4 * qd + 1]), as_u32(s[4 * qd + 2]), as_u32(s[4 * qd + 3])};
#pragma unroll
      for (int db = 0; db < C::kDB; ++db)
        mfma_step<float>(*reinterpret_cast<const u32x4*>(vt + ((db * 32 + r) * kNarrowVS + 8 * qd + 4 * g) * 4 + db * kNarrowShift), pf, o[db]);
    }
  };

  for (int blk = wave; blk < nblk; blk += C::kSets * NW) {
    step(blk, kfa, vra);
    if (C::kSets == 2 && blk + NW < nblk) step(blk + NW, kfb, vrb);
  }

  // ---- merge the waves' partial results through LDS (the V tiles are no longer needed)
  const float l_tot = sum_halves(l);
  float* mo = reinterpret_cast<float*>(smem);                          // [wave][db][i][lane]
  float2* ml = reinterpret_cast<float2*>(smem + C::kLds - NW * 32 * 8);  // [wave][query]
  __syncthreads();
#pragma unroll
  for (int db = 0; db < C::kDB; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) mo[((wave * C::kDB + db) * 16 + i) * 64 + lane] = o[db][i];
  if (g == 0) ml[wave * 32 + r] = make_float2(m, l_tot);
  __syncthreads();
  float M = kNegBig;
#pragma unroll
  for (int w = 0; w < NW; ++w) M = fmaxf(M, ml[w * 32 + r].x);
  float wgt[NW];
  float L = 0.f;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    const float2 v = ml[w * 32 + r];
    wgt[w] = fast_exp2(v.x - M);
    L += wgt[w] * v.y;
  }
  if (q >= prm.n_q) return;
  const float inv = 1.f / L;
  char* orow = prm.O.group_row(b, h, prm.q_per_kv, prm.n_resp, q);
  // the kDB * 4 groups of four output elements are dealt over the waves
  for (int item = wave; item < C::kDB * 4; item += NW) {
    const int db = item >> 2, qd = item & 3;
    float v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float acc = 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w) acc += wgt[w] * mo[((w * C::kDB + db) * 16 + 4 * qd + e) * 64 + lane];
      v[e] = acc * inv;
    }
    char* to = orow + (db * 32 + 8 * qd + 4 * g) * C::kEB;
    *reinterpret_cast<float4*>(to) = make_float4(v[0], v[1], v[2], v[3]);
  }
  if (prm.lse && wave == 0 && g == 0) prm.lse[(int64_t)bh * prm.n_q + q] = (M + __log2f(L)) * kLn2;
}

typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;

// fp32 in pieces of 16 queries and 16 keys: eight waves a workgroup, two blocks in flight a wave, no LDS before the merge.  For launches
// that leave compute units without a workgroup of 32 queries: what bounds these is a wave's own chain, of which the products of a
// block of 32 x 32 are 4096 cycles (head_dim 64) on one wave, and here 1024.  The elements of a row are taken in an
// order in which a lane's operands are 16 consecutive bytes: in the logits' k-step 4t + e lane group g has element 16t + 4g + e of K and
// Q; of V lane c has elements 4c .. 4c+3 of key 4g + i, one for each of four tiles of O^T, and the probabilities are the other operand
// as they come.
template <int D>
struct SmallCfg {
  static constexpr int kWaves = 8, kThreads = 64 * kWaves;
  static constexpr int kQ = 16, kKeys = 16;
  static constexpr int kRowB = 4 * D;
  static constexpr int kChunks = D / 16;        // 16-byte pieces of a row of K or Q per lane
  static constexpr int kHalves = D / 64;        // tiles of O^T, in fours
  static constexpr int kRowP = kRowB + 16;      // a row of partial O in LDS
  static constexpr int kOffMl = kWaves * kQ * kRowP;
  static constexpr int kLds = kOffMl + kWaves * kQ * 8;
};

__device__ __forceinline__ float max_of_groups(float v) {  // over the lanes c, c + 16, c + 32, c + 48
  const auto sw = __builtin_amdgcn_permlane16_swap(as_u32(v), as_u32(v), false, false);
  const unsigned u0 = sw[0], u1 = sw[1];
  v = fmaxf(as_f32(u0), as_f32(u1));
  return max_halves(v);
}
__device__ __forceinline__ float sum_of_groups(float v) {
  const auto sw = __builtin_amdgcn_permlane16_swap(as_u32(v), as_u32(v), false, false);
  const unsigned u0 = sw[0], u1 = sw[1];
  v = as_f32(u0) + as_f32(u1);
  return sum_halves(v);
}

template <int D>
__global__ __launch_bounds__(SmallCfg<D>::kThreads) void attend_small_kernel(const AttendParams prm) {
  fetch_attend_arguments<true>();
  using C = SmallCfg<D>;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;
  const int nqt = (prm.n_q + C::kQ - 1) / C::kQ;
  // eight runs of consecutive (head, query tile) pairs, one per XCD
  const int pair = (blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8;
  const int bh = pair / nqt;
  const int qt = pair - bh * nqt;
  if (bh >= prm.BH) return;
  const int b = bh / prm.H;
  const int h = bh - b * prm.H;
  const int lane = threadIdx.x & 63, c = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int64_t cu0 = 0, cu1 = 0;
  if (!prm.full) {
    const auto cu = (const __attribute__((address_space(4))) int32_t*)(prm.cu + bh);
    cu0 = cu[0];
    cu1 = cu[1];
  }
  const int n2 = prm.n_resp + (prm.full ? prm.lens.P[b] : 0);  // rows of the second segment

  const int nb2 = (n2 + C::kKeys - 1) / C::kKeys;
  struct Block {
    f32x4 k[C::kChunks], v[C::kHalves][4];
  };
  // Rows past the end of a segment re-read its last row; their logits are masked and their values zeroed.
  auto load = [&](const char* k, int64_t kst, const char* v, int64_t vst, int last, Block& to) {
    const char* krow = k + min(c, last) * kst + g * 16;
#pragma unroll
    for (int t = 0; t < C::kChunks; ++t) to.k[t] = *reinterpret_cast<const f32x4*>(krow + t * 64);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const char* vrow = v + min(4 * g + i, last) * vst + c * 16;
#pragma unroll
      for (int half = 0; half < C::kHalves; ++half) to.v[half][i] = *reinterpret_cast<const f32x4*>(vrow + half * 256);
    }
  };
  const char *k2 = prm.K2.row(b, h, 0), *v2 = prm.V2.row(b, h, 0);
  auto resp = [&](int t, Block& to) {
    const int first = t * C::kKeys;
    load(k2 + first * prm.K2.stride_t, prm.K2.stride_t, v2 + first * prm.V2.stride_t, prm.V2.stride_t, n2 - 1 - first, to);
  };
  Block one, two;
  // (the response segment comes first: its blocks are asked for before the head's budget is known)
  if (wave < nb2) resp(wave, one);
  f32x4 qf[C::kChunks];
  {
    const char* qrow = prm.Q.group_row(b, h, prm.q_per_kv, prm.n_resp, min(qt * C::kQ + c, prm.n_q - 1)) + g * 16;
#pragma unroll
    for (int t = 0; t < C::kChunks; ++t) qf[t] = *reinterpret_cast<const f32x4*>(qrow + t * 64);
  }
  const int64_t c0 = min(cu0, prm.capacity);
  const int len_a = (int)(min(cu1, prm.capacity) - c0);
  const char *a_k = prm.Kc + c0 * C::kRowB, *a_v = prm.Vc + c0 * C::kRowB;
  const int nblk = nb2 + (len_a + C::kKeys - 1) / C::kKeys;
  auto ask = [&](int t, Block& to) {
    if (t < nb2) {
      resp(t, to);
    } else {
      const int64_t first = (int64_t)(t - nb2) * C::kKeys;
      load(a_k + first * C::kRowB, C::kRowB, a_v + first * C::kRowB, C::kRowB, len_a - 1 - (int)first, to);
    }
  };
  if (wave >= nb2 && wave < nblk) ask(wave, one);
  if (wave + C::kWaves < nblk) ask(wave + C::kWaves, two);

  f32x4 o[C::kHalves][4];
#pragma unroll
  for (int half = 0; half < C::kHalves; ++half)
#pragma unroll
    for (int t = 0; t < 4; ++t) o[half][t] = f32x4{};
  float m = kNegBig, l = 0.f;
  auto step = [&](int t, Block& of) {
    // S^T = K Q^T: this lane's keys are 4g .. 4g+3 of the block, its query is c
    f32x4 s = f32x4{}, s1 = f32x4{};
#pragma unroll
    for (int p = 0; p < C::kChunks; ++p)
#pragma unroll
      for (int e = 0; e < 4; e += 2) {
        s = __builtin_amdgcn_mfma_f32_16x16x4f32(of.k[p][e], qf[p][e], s, 0, 0, 0);
        s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(of.k[p][e + 1], qf[p][e + 1], s1, 0, 0, 0);
      }
    s += s1;
    const int valid = t < nb2 ? n2 - t * C::kKeys : len_a - (t - nb2) * C::kKeys;
    if (valid < C::kKeys) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (4 * g + i >= valid) {
          s[i] = -INFINITY;
#pragma unroll
          for (int half = 0; half < C::kHalves; ++half) of.v[half][i] = f32x4{};
        }
    }
    // online softmax, the reference raised lazily as in the tiled kernel
    const float cand = max_of_groups(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]))) * prm.c;
    const bool bump = cand > m + kLazyBump;
    if (__any(bump)) {
      const float m_new = bump ? cand : m;
      const float alpha = fast_exp2(m - m_new);
      m = m_new;
      l *= alpha;
#pragma unroll
      for (int half = 0; half < C::kHalves; ++half)
#pragma unroll
        for (int u = 0; u < 4; ++u) o[half][u] *= alpha;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      s[i] = fast_exp2(fmaf(s[i], prm.c, -m));
      l += s[i];
    }
    // O^T += V^T P^T: row r of tile u is element 4r + u
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int half = 0; half < C::kHalves; ++half)
#pragma unroll
        for (int u = 0; u < 4; ++u) o[half][u] = __builtin_amdgcn_mfma_f32_16x16x4f32(of.v[half][i][u], s[i], o[half][u], 0, 0, 0);
    if (t + 2 * C::kWaves < nblk) ask(t + 2 * C::kWaves, of);
  };
  for (int t = wave; t < nblk; t += 2 * C::kWaves) {
    step(t, one);
    if (t + C::kWaves < nblk) step(t + C::kWaves, two);
  }

  // ---- the waves' partial results through LDS, by rows
  const float l_tot = sum_of_groups(l);
#pragma unroll
  for (int half = 0; half < C::kHalves; ++half)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      *in_lds<f32x4>(lds0 + (wave * C::kQ + c) * C::kRowP + g * 64, half * 256 + i * 16) = f32x4{o[half][0][i], o[half][1][i], o[half][2][i], o[half][3][i]};
  if (g == 0) *in_lds<f32x2>(lds0 + C::kOffMl + (wave * C::kQ + c) * 8) = f32x2{m, l_tot};
  __syncthreads();
  const int row = (int)threadIdx.x / (D / 4), piece = (int)threadIdx.x % (D / 4);
  const int q = qt * C::kQ + row;
  if (row >= C::kQ || q >= prm.n_q) return;
  f32x2 ml[C::kWaves];
  f32x4 part[C::kWaves];
#pragma unroll
  for (int w = 0; w < C::kWaves; ++w) {
    ml[w] = *in_lds<const f32x2>(lds0 + C::kOffMl + row * 8, w * C::kQ * 8);
    part[w] = *in_lds<const f32x4>(lds0 + row * C::kRowP + piece * 16, w * C::kQ * C::kRowP);
  }
  float top = kNegBig, L = 0.f;
#pragma unroll
  for (int w = 0; w < C::kWaves; ++w) top = fmaxf(top, ml[w][0]);
  f32x4 acc = f32x4{};
#pragma unroll
  for (int w = 0; w < C::kWaves; ++w) {
    const float weight = fast_exp2(ml[w][0] - top);
    L += weight * ml[w][1];
    acc += weight * part[w];
  }
  acc *= 1.f / L;
  *reinterpret_cast<f32x4*>(prm.O.group_row(b, h, prm.q_per_kv, prm.n_resp, q) + piece * 16) = acc;
  if (prm.lse && piece == 0) prm.lse[(int64_t)bh * prm.n_q + q] = (top + __log2f(L)) * kLn2;
}

// bf16: eight waves, 32 queries, K, V and the queries by direct transfers into LDS (a load of K fragments touches 32 rows for
// 1 KiB), V read with transposing loads.  A wave has one block in flight: the next K is asked for once the logits are formed, the
// next V once the block is added, and each is waited for on its own (the compiler, which does not see the transfers, would wait
// for later ones as well).  The key axis begins with the response segment, whose blocks are asked for before the head's budget is known.
// The partial results are merged by rows, so that 16 threads write a row in whole pieces.
//
// What bounds it: the latency of each round of blocks, 1.5 us for loads at about the rate of L2 and the arithmetic of two waves a SIMD;
// 32 heads x 256 queries x 512 keys take 9.3 us: 1.8 for an empty launch, 2.1 until the first blocks are there, 1.0 and 1.5 per
// round, 1.2 for the merge.  Before, four waves with K straight into registers and two blocks in flight 10.9 (13.7 against 9.3 in a
// layer over 4k tokens, where K and V are not in L2); four waves with K by transfers 11.5, the merge with each lane writing the 8 bytes
// of its accumulators 10.2.
//
// The reference is raised with every new maximum of a wave, not lazily: a row's largest probabilities are then powers of two, which
// bf16 holds without rounding, whichever segment they come from.  Raised lazily by response blocks that come first, it left the larger
// probabilities of the kept rows behind them with a rounding each: errors of O against 64 bits 8 to 25 % above those of a kernel
// that took the kept rows first (32 heads x 256 queries over 128 + 256 keys 2.26e-3 and 1.81e-3, now 1.78e-3).  It costs a rescaling in
// most blocks: over 512 keys 8.6 -> 8.7 us, 8 heads x 256 queries x 3256 keys 24.2 -> 25.1 (with the other kernel 10.6 and 33.8).
template <int D>
struct PairsCfg {
  static constexpr int kWaves = 8, kThreads = 64 * kWaves;
  static constexpr int kRowB = 2 * D;
  static constexpr int kSteps = kRowB / 32;
  static constexpr int kPPR = kRowB / 16;        // 16-byte pieces per row
  static constexpr int kRPI = 1024 / kRowB;      // rows moved by one transfer
  static constexpr int kMoves = 32 / kRPI;       // transfers of a block
  static constexpr int kDB = D / 32;
  static constexpr int kBlock = 32 * kRowB;
  static constexpr int kWaveB = 2 * kBlock;      // K and V of a wave's block; at the end its partial O
  static constexpr int kOffQ = kWaves * kWaveB;
  static constexpr int kOffMl = kOffQ + kBlock;  // [wave][query] (m, l)
  static constexpr int kLds = kOffMl + kWaves * 32 * 8;
  // Piece p of row r of K or Q is in slot p ^ swz(r): the fragments of 16 consecutive rows are on different banks.
  static __device__ constexpr uint32_t swz(uint32_t row) { return D == 128 ? row & 15 : (row >> 1) & 7; }
};

template <int D>
__global__ __launch_bounds__(PairsCfg<D>::kThreads) void attend_pairs_kernel(const AttendParams prm) {
  fetch_attend_arguments<true>();
  using C = PairsCfg<D>;
  constexpr int S = C::kSteps, M = C::kMoves;
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;

  const int nqt = (prm.n_q + 31) / 32;
  // eight runs of consecutive (head, query tile) pairs, one per XCD
  const int pair = (blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8;
  const int bh = pair / nqt;
  const int qt = pair - bh * nqt;
  if (bh >= prm.BH) return;
  const int b = bh / prm.H;
  const int h = bh - b * prm.H;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane & 31;
  const int g = lane >> 5;
  int64_t cu0 = 0, cu1 = 0;
  if (!prm.full) {
    const auto cu = (const __attribute__((address_space(4))) int32_t*)(prm.cu + bh);
    cu0 = cu[0];
    cu1 = cu[1];
  }
  const int n2 = prm.n_resp + (prm.full ? prm.lens.P[b] : 0);  // rows of the second segment

  // Rows past the end of a segment re-read its last row and are masked.
  const uint32_t mrow = (uint32_t)lane / C::kPPR, slot = (uint32_t)lane % C::kPPR;
  const uint32_t vpiece = (slot ^ v_swizzle<D>(mrow) << 1) << 4;
  const uint32_t own = lds0 + wave * C::kWaveB;
  auto move = [&](const char* base, uint32_t st, int last, bool k, uint32_t to) {
    auto piece = [&](int i) { return k ? (slot ^ C::swz(mrow) ^ C::swz(i * C::kRPI)) << 4 : vpiece; };
    if (last >= 31) {
      const uint32_t off = mrow * st;
#pragma unroll
      for (int i = 0; i < M; ++i) dma16(base + (int64_t)(i * C::kRPI) * st, off + piece(i), to + i * 1024);
    } else {
#pragma unroll
      for (int i = 0; i < M; ++i) dma16(base, (uint32_t)min(i * C::kRPI + (int)mrow, last) * st + piece(i), to + i * 1024);
    }
  };
  const int nb2 = (n2 + 31) / 32;
  const char *k2 = prm.K2.row(b, h, 0), *v2 = prm.V2.row(b, h, 0);
  const uint32_t kst = (uint32_t)prm.K2.stride_t, vst = (uint32_t)prm.V2.stride_t;

  // this wave's part of the queries, then its first blocks
  {
#pragma unroll
    for (int j = wave; j < M; j += C::kWaves) {
      const char* qrow = prm.Q.group_row(b, h, prm.q_per_kv, prm.n_resp, min(qt * 32 + j * C::kRPI + (int)mrow, prm.n_q - 1));
      dma16_from(qrow + ((slot ^ C::swz(j * C::kRPI + mrow)) << 4), lds0 + C::kOffQ + j * 1024);
    }
  }
  auto resp_k = [&](int t) { move(k2 + (int64_t)(t * 32) * kst, kst, n2 - 1 - t * 32, true, own); };
  auto resp_v = [&](int t) { move(v2 + (int64_t)(t * 32) * vst, vst, n2 - 1 - t * 32, false, own + C::kBlock); };
  if (wave < nb2) {
    resp_k(wave);
    resp_v(wave);
  }
  const int64_t c0 = min(cu0, prm.capacity);
  const int len_a = (int)(min(cu1, prm.capacity) - c0);
  const char *a_k = prm.Kc + c0 * C::kRowB, *a_v = prm.Vc + c0 * C::kRowB;
  const int nblk = nb2 + (len_a + 31) / 32;
  auto ask_k = [&](int t) {
    if (t < nb2)
      resp_k(t);
    else
      move(a_k + (int64_t)((t - nb2) * 32) * C::kRowB, C::kRowB, len_a - 1 - (t - nb2) * 32, true, own);
  };
  auto ask_v = [&](int t) {
    if (t < nb2)
      resp_v(t);
    else
      move(a_v + (int64_t)((t - nb2) * 32) * C::kRowB, C::kRowB, len_a - 1 - (t - nb2) * 32, false, own + C::kBlock);
  };
  if (wave >= nb2 && wave < nblk) {
    ask_k(wave);
    ask_v(wave);
  }
  // the queries are there: only the block may be on its way
  if (wave < nblk)
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"i"(2 * M) : "memory");
  else
    asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
  uint32_t fa[S];  // this lane's pieces of row r
  u32x4 qf[S];
#pragma unroll
  for (int s = 0; s < S; ++s) {
    fa[s] = r * C::kRowB + (((2 * s + g) ^ C::swz(r)) << 4);
    qf[s] = *in_lds<const u32x4>(lds0 + C::kOffQ + fa[s]);
    fa[s] += own;
  }
  uint32_t va[C::kDB];  // this lane's transposing reads of a V block
#pragma unroll
  for (int db = 0; db < C::kDB; ++db) va[db] = own + C::kBlock + v_read_offset<D>(lane, db);

  f32x16 o[C::kDB];
#pragma unroll
  for (int db = 0; db < C::kDB; ++db) o[db] = f32x16{};
  float m = kNegBig, l = 0.f;
  const float c = prm.c;
  for (int t = wave; t < nblk; t += C::kWaves) {
    const bool more = t + C::kWaves < nblk;
    asm volatile("s_waitcnt vmcnt(%0)" ::"i"(M) : "memory");  // K is there, V may be on its way
    // S^T = K Q^T: keys on rows, queries on columns
    f32x16 s = f32x16{};
#pragma unroll
    for (int st = 0; st < S; ++st) {
      const u32x4 kf = *in_lds<const u32x4>(fa[st]);
      mfma_step<bf16_t>(kf, qf[st], s);
    }
    asm volatile("" : "+v"(s) : : "memory");  // (the slot has been read)
    if (more) ask_k(t + C::kWaves);
    const int valid = t < nb2 ? n2 - t * 32 : len_a - (t - nb2) * 32;
    if (valid < 32) {
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (8 * (i / 4) + 4 * g + (i % 4) >= valid) s[i] = -INFINITY;
    }
    // online softmax; lanes l and l^32 hold the same query
    float bm = s[0];
#pragma unroll
    for (int i = 1; i < 16; ++i) bm = fmaxf(bm, s[i]);
    bm = max_halves(bm);
    const float cand = bm * c;
    const bool bump = cand > m;  // (each time, see above)
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
    for (int i = 0; i < 16; ++i) {
      const float pv = fast_exp2(fmaf(s[i], c, -m));
      s[i] = pv;
      psum += pv;
    }
    l += psum;
    if (more)
      asm volatile("s_waitcnt vmcnt(%0)" ::"i"(M) : "memory");
    else
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (valid < 32) {  // (rows that do not exist: zero times an infinity of the row that was read instead is no zero)
      for (int i = valid * C::kPPR + lane; i < 32 * C::kPPR; i += 64) *in_lds<u32x4>(own + i * 16, C::kBlock) = u32x4{0u, 0u, 0u, 0u};
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
    // O^T += V^T P^T
#pragma unroll
    for (int tp = 0; tp < 2; ++tp) {
      u32x4 pf;
#pragma unroll
      for (int w = 0; w < 4; ++w) pf[w] = pack_bf16x2(s[8 * tp + 2 * w], s[8 * tp + 2 * w + 1]);
#pragma unroll
      for (int db = 0; db < C::kDB; ++db) {
        const int imm = 16 * tp * C::kRowB;
        const u32x2 lo = read_transposed(va[db], imm), hi = read_transposed(va[db], imm + 8 * C::kRowB);
        const u32x4 vf = {lo[0], lo[1], hi[0], hi[1]};
        mfma_step<bf16_t>(vf, pf, o[db]);
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the slot has been read
    if (more) ask_v(t + C::kWaves);
  }

  // ---- the waves' partial results, each in its wave's own LDS: four elements of O^T at a time, group k = d / 8 of a query and half
  // g = d / 4 % 2 in slot (query + 32 g) ^ mix(k, g) of 64, so that a row's pieces, which its threads read next, are on different banks
  constexpr int kPieces = D / 64;  // of four elements a thread, side by side
  auto mix = [](int k, int g) { return D == 128 ? k : k ^ g << 3; };
  const float l_tot = sum_halves(l);
#pragma unroll
  for (int k = 0; k < D / 8; ++k)
    *in_lds<f32x4>(own + ((lane ^ mix(k, g)) << 4), k * 1024) = f32x4{o[k / 4][k % 4 * 4], o[k / 4][k % 4 * 4 + 1], o[k / 4][k % 4 * 4 + 2], o[k / 4][k % 4 * 4 + 3]};
  if (g == 0) *in_lds<f32x2>(lds0 + C::kOffMl + (wave * 32 + r) * 8) = f32x2{m, l_tot};
  __syncthreads();
  const int row = (int)threadIdx.x / 16, p0 = (int)threadIdx.x % 16 * kPieces;  // (16 threads a row)
  f32x2 ml[C::kWaves];
  f32x4 part[kPieces][C::kWaves];
#pragma unroll
  for (int w = 0; w < C::kWaves; ++w) ml[w] = *in_lds<const f32x2>(lds0 + C::kOffMl + row * 8, w * 32 * 8);
#pragma unroll
  for (int i = 0; i < kPieces; ++i) {
    const int k = (p0 + i) / 2, half = (p0 + i) % 2;
    const uint32_t from = lds0 + k * 1024 + (((row + 32 * half) ^ mix(k, half)) << 4);
#pragma unroll
    for (int w = 0; w < C::kWaves; ++w) part[i][w] = *in_lds<const f32x4>(from, w * C::kWaveB);
  }
  float top = kNegBig, L = 0.f, wgt[C::kWaves];
#pragma unroll
  for (int w = 0; w < C::kWaves; ++w) top = fmaxf(top, ml[w][0]);
#pragma unroll
  for (int w = 0; w < C::kWaves; ++w) {
    wgt[w] = fast_exp2(ml[w][0] - top);
    L += wgt[w] * ml[w][1];
  }
  const int q = qt * 32 + row;
  if (q >= prm.n_q) return;
  const float inv = 1.f / L;
  uint32_t out[2 * kPieces];
#pragma unroll
  for (int i = 0; i < kPieces; ++i) {
    f32x4 v = wgt[0] * part[i][0];
#pragma unroll
    for (int w = 1; w < C::kWaves; ++w) v += wgt[w] * part[i][w];
    out[2 * i] = pack_bf16x2(v[0] * inv, v[1] * inv);
    out[2 * i + 1] = pack_bf16x2(v[2] * inv, v[3] * inv);
  }
  char* to = prm.O.group_row(b, h, prm.q_per_kv, prm.n_resp, q) + p0 * 8;
  if constexpr (kPieces == 2)
    *reinterpret_cast<u32x4*>(to) = u32x4{out[0], out[1], out[2], out[3]};
  else
    *reinterpret_cast<u32x2*>(to) = u32x2{out[0], out[1]};
  if (prm.lse && p0 == 0) prm.lse[(int64_t)bh * prm.n_q + q] = (top + __log2f(L)) * kLn2;
}

// Merge the key splits of the query rows: O = sum_s w_s O_s / sum_s w_s l_s, w_s = 2^(m_s - max m).
// A row is served by D/4 consecutive threads (four output elements each, 16-byte loads of the partials).
// N splits' partials are asked for before the first is used, as the waits are what it takes its time for.  Two splits need N = 2, more of
// them 4 or 8 (us before, each loop waiting for its loads, and now: 2 splits of 16 x 506 rows 8.9 / 7.3, 64 x 106 rows, 8 splits, 6.9 / 4.8,
// 4 x 265 rows, 20 splits, 12.2 / 6.4; with eight asked for where there are two 7.4 and, 96 x 148 rows, 5.6 for 5.3).
template <typename T, int D, int N>
__global__ __launch_bounds__(256) void attend_merge_kernel(const AttendParams prm) {
  fetch_arguments({MASKKV_VIEW_ARGUMENTS(AttendParams, O), MASKKV_ARGUMENT(AttendParams, H), MASKKV_ARGUMENT(AttendParams, part_ml)});
  constexpr int kTPR = D / 4;          // threads per row
  constexpr int kRows = 256 / kTPR;    // rows per workgroup
  const int bh = blockIdx.y;
  const int b = bh / prm.H, h = bh % prm.H;
  const int q = blockIdx.x * kRows + (int)threadIdx.x / kTPR;
  const int e = ((int)threadIdx.x % kTPR) * 4;
  if (q >= prm.n_q) return;
  const float2* ml_of = prm.part_ml + (int64_t)bh * prm.n_splits * prm.n_q + q;
  const float* o_of = prm.part_o + ((int64_t)bh * prm.n_splits * prm.n_q + q) * D + e;
  float2 ml[N];
  float4 o[N];
  auto ask_ml = [&](int s0) {
#pragma unroll
    for (int u = 0; u < N; ++u)
      if (s0 + u < prm.n_splits) ml[u] = ml_of[(int64_t)(s0 + u) * prm.n_q];
  };
  auto ask_o = [&](int s0) {
#pragma unroll
    for (int u = 0; u < N; ++u)
      if (s0 + u < prm.n_splits) o[u] = *reinterpret_cast<const float4*>(o_of + (int64_t)(s0 + u) * prm.n_q * D);
  };
  ask_ml(0);
  ask_o(0);
  float M = kNegBig;
  for (int s0 = 0; s0 < prm.n_splits; s0 += N) {
    if (s0 > 0) ask_ml(s0);
#pragma unroll
    for (int u = 0; u < N; ++u)
      if (s0 + u < prm.n_splits) M = fmaxf(M, ml[u].x);
  }
  float L = 0.f;
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int s0 = 0; s0 < prm.n_splits; s0 += N) {
    if (prm.n_splits > N) ask_ml(s0);
    if (s0 > 0) ask_o(s0);
#pragma unroll
    for (int u = 0; u < N; ++u)
      if (s0 + u < prm.n_splits) {
        const float w = fast_exp2(ml[u].x - M);
        L += w * ml[u].y;
        acc.x += w * o[u].x;
        acc.y += w * o[u].y;
        acc.z += w * o[u].z;
        acc.w += w * o[u].w;
      }
  }
  const float inv = 1.f / L;
  char* orow = prm.O.group_row(b, h, prm.q_per_kv, prm.n_resp, q);
  if (sizeof(T) == 2) {
    u32x2 w;
    w[0] = pack_bf16x2(acc.x * inv, acc.y * inv);
    w[1] = pack_bf16x2(acc.z * inv, acc.w * inv);
    *reinterpret_cast<u32x2*>(orow + e * 2) = w;
  } else {
    *reinterpret_cast<float4*>(orow + e * 4) = make_float4(acc.x * inv, acc.y * inv, acc.z * inv, acc.w * inv);
  }
  if (prm.lse && e == 0) prm.lse[(int64_t)bh * prm.n_q + q] = (M + __log2f(L)) * kLn2;
}

// Heads by descending key count, for the compressed call of the tiled kernel: budgets are ragged, the hardware
// hands workgroups to compute units in launch order, and the longest heads should not start last (measured
// on 256 heads with 576...1536 keys: 101 us in this order, 123 us in the given order).  A counting sort by
// 64-key tile count in one workgroup; the order inside a bucket is whatever the atomics give, which does not
// matter: every head's result is independent of when it runs.  (fp32, and bf16 with more heads than kRankHeads: up to that number
// the workgroups of the bf16 kernel find their heads themselves.)
constexpr int kOrderThreads = 1024;
constexpr int kOrderBuckets = 1024;

__global__ __launch_bounds__(kOrderThreads) void attend_order_kernel(const int32_t* cu, int64_t capacity, int BH,
                                                                     int n_resp, int32_t* order) {
  __shared__ int count[kOrderBuckets];
  __shared__ int wave_total[kOrderThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  auto bucket_of = [&](int bh) {
    const int64_t c0 = min((int64_t)cu[bh], capacity), c1 = min((int64_t)cu[bh + 1], capacity);
    const int64_t tiles = (c1 - c0 + n_resp + 63) / 64;
    return kOrderBuckets - 1 - (int)min((int64_t)(kOrderBuckets - 1), tiles);  // bucket 0 = longest
  };
  count[tid] = 0;
  __syncthreads();
  for (int bh = tid; bh < BH; bh += kOrderThreads) atomicAdd(&count[bucket_of(bh)], 1);
  __syncthreads();
  // exclusive prefix sum over the buckets, one bucket per thread
  const int mine = count[tid];
  int incl = mine;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int n = __shfl_up(incl, o, 64);
    if (lane >= o) incl += n;
  }
  if (lane == 63) wave_total[wave] = incl;
  __syncthreads();
  int before = 0;
  for (int w = 0; w < wave; ++w) before += wave_total[w];
  count[tid] = before + incl - mine;  // first slot of this bucket
  __syncthreads();
  for (int bh = tid; bh < BH; bh += kOrderThreads) order[atomicAdd(&count[bucket_of(bh)], 1)] = bh;
}

// Queries per workgroup of the tiled kernel for this description.
int tiled_queries(const maskkv_desc* d, bool full) {
  if (d->dtype != MASKKV_BF16) return AttCfg<128>::kQPerBlock;
  return attend_tiles_queries((int64_t)d->B * d->H, d->n_resp * query_heads_per_kv(d), full);
}

int attend_splits(const maskkv_desc* d, bool full) {
  if (!full) return 1;
  const int per_block = tiled_queries(d, full);
  const int64_t qtiles = ((int64_t)d->n_resp * query_heads_per_kv(d) + per_block - 1) / per_block;
  const int64_t blocks = qtiles * d->B * d->H;
  // one workgroup per compute unit, a single round (bf16: 4 heads x 7 tiles of queries are 252 workgroups, not 280)
  int64_t s = d->dtype == MASKKV_BF16 ? kUnits / blocks : (kUnits + blocks - 1) / blocks;
  const int64_t by_len = ((int64_t)d->P_max + d->n_resp + 511) / 512;
  if (s > by_len) s = by_len;
  if (s > 64) s = 64;
  if (s < 1) s = 1;
  return (int)s;
}

// bf16: the narrow kernel's workgroups of 32 queries are all resident at one (head_dim 128) or two (64) a compute unit.  It is used
// as far as that (half a round more at head_dim 64), and for up to two rounds at head_dim 128 where the key axis is short, as far as
// the capacity of the packed rows tells: each workgroup reads all of its head's keys, the tiled kernel's share them among 128 or 256
// queries (us a call, narrow against tiled.  head_dim 128, 256 workgroups: 512 keys 9.3 / 16.8, 3256 keys 33 / 51; 320 to
// 512 workgroups: 32 heads x 280 queries x 536 keys 15.8 / 18.3, 64 x 256 x 512 15.4 / 17.2, 32 x 512 x 1024 22.1 / 23.0, 32 x 512 x
// 1536 28.2 / 28.9, but 64 x 256 x 1756 38 / 34, 32 x 512 x 4512 75 / 66.  head_dim 64, 512 workgroups: 768 keys 10.6 / 15.3,
// 3512 keys 30 / 42; 640: 2140 keys 26.8 / 29.3; 768: 1024 keys 17.1 / 18.0, 3768 keys 45.6 / 45.2; 1024: 768 keys 18.5 / 16.1.)
// fp32: a round of narrow workgroups takes a quarter (head_dim 64) to a seventh (128) of a round of the tiled kernel's, whose eight
// waves walk the whole key axis (32 heads x 256 queries x 512 keys: 16.8 / 75 and 29.5 / 143 us; 4 heads x 64 queries x 576 keys
// 18.7 / 78.6), so it is taken up to four times as many rounds.
bool attend_is_narrow(const maskkv_desc* d, bool full, int64_t capacity) {
  if (full) return false;
  const int64_t n_q = (int64_t)d->n_resp * query_heads_per_kv(d), heads = (int64_t)d->B * d->H;
  const int64_t groups = (n_q + 31) / 32 * heads;
  if (d->dtype == MASKKV_BF16) {
    if (d->d == 64) return groups <= 5 * kUnits / 2;
    return groups <= kUnits || (groups <= 2 * kUnits && capacity / heads <= 1280 - d->n_resp);  // (capacity may be any int64_t)
  }
  const int64_t tiled = (n_q + AttCfg<128>::kQPerBlock - 1) / AttCfg<128>::kQPerBlock * heads;
  return groups <= 4 * kUnits * ((tiled + kUnits - 1) / kUnits);
}

// fp32: workgroups of 16 queries as long as there is one a compute unit at most (us a call, against the narrow kernel's 32: 4 heads x 64
// queries x 96 keys, head_dim 64, 6.1 / 7.7; 12 x 73 x 273, head_dim 128, 12.7 / 21.8; 16 x 256 x 512 11.4 / 16.8 and 19.2 / 27.3; but
// 20 x 256 x 512 18.9 / 16.6 and 33.9 / 27.3, 32 x 512 x 2512 256 / 209).
bool attend_is_small(const maskkv_desc* d) {
  const int64_t n_q = (int64_t)d->n_resp * query_heads_per_kv(d);
  return (n_q + 15) / 16 * d->B * d->H <= kUnits;
}

// The un-evicted call of few query tiles over a short prompt: one of the narrow kernels instead of a tiled one on splits of the key axis and a
// merge, as long as the key axis, which each of their workgroups walks alone, is not too long for the launch (us a call,
// narrow / tiled.  bf16, head_dim 128: 4 heads x 64 queries, 1064 keys 11 / 17, 3064 21 / 21; 32 x 256, 1256 14 / 29, 5256
// 42 / 45, 8256 65 / 56; 64 x 256, 1256 26 / 30, 3256 59 / 50; head_dim 64: 4 x 64, 3064 15.5 / 17.0, 5064 22 / 19; 32 x 256, 8256 35 / 38; 32 x 400,
// 5400 38 / 41, 8400 56 / 55.  fp32, 16 queries a workgroup: 4 x 36, head_dim 128, 336 keys 14 / 94, 2936 74 / 141; 16 x 256, head_dim 64,
// 3156 42 / 80; 32: 32 x 256, 2900 + 256 keys 76 / 82 and 140 / 148, 32 x 512, 1512 70 / 80 and 139 / 152, 3412 143 / 131 and 296 / 246.)
bool attend_full_is_narrow(const maskkv_desc* d, const Lens& lens) {
  const int64_t n_q = (int64_t)d->n_resp * query_heads_per_kv(d), groups = (n_q + 31) / 32 * d->B * d->H;
  int64_t keys = 0;
  for (int b = 0; b < d->B; ++b) keys = max(keys, (int64_t)lens.P[b] + d->n_resp);
  if (d->dtype == MASKKV_BF16) {
    const bool wide = d->d == 128;
    if (groups <= kUnits) return keys <= (wide ? 2700 + 10 * groups : 3800 + 20 * groups);
    return groups <= 2 * kUnits && keys <= (wide ? 1800 : 5000);
  }
  if (attend_is_small(d)) return keys <= 5000;
  return groups <= kUnits ? keys <= 3200 : groups <= 2 * kUnits && keys <= 1500;
}

constexpr int64_t kCacheBytes = (int64_t)256 << 20;  // of the memory-side cache

// Heads are only put in order where not every workgroup of the tiled kernel starts at once.
bool attend_is_ordered(const maskkv_desc* d, bool full, int64_t capacity) {
  if (full || attend_is_narrow(d, full, capacity)) return false;
  const int per_block = tiled_queries(d, full);
  return ((int64_t)d->n_resp * query_heads_per_kv(d) + per_block - 1) / per_block * d->B * d->H > kUnits;
}

// The un-evicted call's V passes by the memory-side cache where it is read once (one tile of queries) and K and V together are larger
// than that cache: V would push out K, which the scoring that follows reads again.  (us for this call and scoring with its normalisers, 32 heads x
// 256 queries, head_dim 128, with it and without, in a loop over the same tensors; over four sets of them in turn: 9k keys 86.3 / 84.6;
// 90.9 / 91.4, 13k 106.4 / 105.3; 113.6 / 114.1, 16k 123.3 / 125.3; 133.5 / 134.7, 20k 144.6 / 150.5; 155.0 / 155.5, 26k 180 / 191; 190.5 / 194.9,
// 33k 226 / 240; 235.9 / 240.3, 48k 328 / 335; 335 / 338.  K as well: 242 / 244 at 33k keys.  Scoring from the last key to the first: the same.
// This call alone: 17k 79 / 84; 85 / 85, 20k 90 / 96; 97 / 97, 26k 112 / 121; 121 / 122, 33k 147 / 149; 148 / 149; with 128 queries 17k 54.5 / 56;
// 63 / 65, 26k 77 / 90; 86 / 90; head_dim 64, 34k 97 / 102; 101 / 101, 40k 112 / 118; 118 / 118, with 128 queries 68 / 73; 73 / 74; 4 sequences of
// 5k 95 / 102; 102 / 103.)
bool attend_is_streamed(const maskkv_desc* d, const Lens& lens, bool full) {
  if (!full || d->n_resp * query_heads_per_kv(d) > tiled_queries(d, true)) return false;
  int64_t keys = 0;
  for (int b = 0; b < d->B; ++b) keys += lens.P[b] + d->n_resp;
  return keys * d->H * d->d * 4 > kCacheBytes;
}

template <int D>
int launch_attend_narrow(const AttendParams& prm, hipStream_t stream) {
  using C = NarrowCfg<D>;
  static bool raised = false;  // one-time opt-in to more than the default dynamic LDS size
  if (C::kLds > 48 * 1024 && !raised) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&attend_narrow_kernel<D>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, C::kLds);
    if (e != hipSuccess) {
      set_error("attend: cannot raise dynamic LDS limit: %s", hipGetErrorString(e));
      (void)hipGetLastError();
      return MASKKV_EHIP;
    }
    raised = true;
  }
  const int nqt = (prm.n_q + 31) / 32;
  const int groups = (prm.BH * nqt + 7) / 8 * 8;
  hipLaunchKernelGGL((attend_narrow_kernel<D>), dim3(groups), dim3(C::kThreads), C::kLds, stream, prm);
  return check_launch("attend (narrow)");
}

template <int D>
int launch_attend_small(const AttendParams& prm, hipStream_t stream) {
  using C = SmallCfg<D>;
  static bool raised = false;  // one-time opt-in to more than the default dynamic LDS size
  if (C::kLds > 48 * 1024 && !raised) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&attend_small_kernel<D>), hipFuncAttributeMaxDynamicSharedMemorySize, C::kLds);
    if (e != hipSuccess) {
      set_error("attend: cannot raise dynamic LDS limit: %s", hipGetErrorString(e));
      (void)hipGetLastError();
      return MASKKV_EHIP;
    }
    raised = true;
  }
  const int groups = (prm.BH * ((prm.n_q + C::kQ - 1) / C::kQ) + 7) / 8 * 8;
  hipLaunchKernelGGL((attend_small_kernel<D>), dim3(groups), dim3(C::kThreads), C::kLds, stream, prm);
  return check_launch("attend (small)");
}

template <int D>
int launch_attend_pairs(const AttendParams& prm, hipStream_t stream) {
  using C = PairsCfg<D>;
  static bool raised = false;  // one-time opt-in to more than the default dynamic LDS size
  if (!raised) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&attend_pairs_kernel<D>), hipFuncAttributeMaxDynamicSharedMemorySize, C::kLds);
    if (e != hipSuccess) {
      set_error("attend: cannot raise dynamic LDS limit: %s", hipGetErrorString(e));
      (void)hipGetLastError();
      return MASKKV_EHIP;
    }
    raised = true;
  }
  const int groups = (prm.BH * ((prm.n_q + 31) / 32) + 7) / 8 * 8;
  hipLaunchKernelGGL((attend_pairs_kernel<D>), dim3(groups), dim3(C::kThreads), C::kLds, stream, prm);
  return check_launch("attend (narrow)");
}

template <typename T, int D>
int launch_attend_t(const AttendParams& prm, int B, hipStream_t stream) {
  using C = AttCfg<D>;
  const int per_block = sizeof(T) == 2 ? attend_tiles_queries((int64_t)B * prm.H, prm.n_q, prm.full) : C::kQPerBlock;
  const int64_t qtiles = (prm.n_q + per_block - 1) / per_block;
  const int64_t units = ((int64_t)B * prm.H * prm.n_splits + 7) / 8 * 8;  // (head, split) pairs, whole rounds of XCDs
  if (units * qtiles > 0x7FFFFFFF) {
    set_error("attend: %lld workgroups exceed the launch limit", (long long)(units * qtiles));
    return MASKKV_ESHAPE;
  }
  if (prm.order) {
    hipLaunchKernelGGL(attend_order_kernel, dim3(1), dim3(kOrderThreads), 0, stream, prm.cu, prm.capacity, prm.BH,
                       prm.n_resp, const_cast<int32_t*>(prm.order));
    if (int e = check_launch("attend (order)")) return e;
  }
  if constexpr (sizeof(T) == 2) {
    if (int e = launch_attend_tiles(prm, D, per_block, stream)) return e;
  } else {
    static bool raised = false;  // one-time opt-in to more than the default dynamic LDS size
    if (C::kLds > 48 * 1024 && !raised) {
      const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&attend_kernel<D>),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, C::kLds);
      if (e != hipSuccess) {
        set_error("attend: cannot raise dynamic LDS limit: %s", hipGetErrorString(e));
        (void)hipGetLastError();
        return MASKKV_EHIP;
      }
      raised = true;
    }
    hipLaunchKernelGGL((attend_kernel<D>), dim3((unsigned)(units * qtiles)), dim3(C::kThreads), C::kLds, stream,
                       prm);
    if (int e = check_launch("attend")) return e;
  }
  if (prm.n_splits > 1) {
    constexpr int kRows = 256 / (D / 4);
    const dim3 grid((prm.n_q + kRows - 1) / kRows, B * prm.H);
    if (prm.n_splits <= 2)
      hipLaunchKernelGGL((attend_merge_kernel<T, D, 2>), grid, dim3(256), 0, stream, prm);
    else if (prm.n_splits <= 4)
      hipLaunchKernelGGL((attend_merge_kernel<T, D, 4>), grid, dim3(256), 0, stream, prm);
    else
      hipLaunchKernelGGL((attend_merge_kernel<T, D, 8>), grid, dim3(256), 0, stream, prm);
    return check_launch("attend merge");
  }
  return MASKKV_OK;
}

}  // namespace

size_t attend_workspace_bytes(const maskkv_desc* d, bool full) {
  const int s = attend_splits(d, full);
  if (!full) return attend_is_ordered(d, full, INT64_MAX) ? ((size_t)d->B * d->H * sizeof(int32_t) + 255) / 256 * 256 : 0;
  if (s == 1) return 0;
  const size_t rows = (size_t)d->B * d->H * s * d->n_resp * query_heads_per_kv(d);
  return (rows * d->d * sizeof(float) + 255) / 256 * 256 + rows * sizeof(float2);
}

int launch_attend(const maskkv_desc* d, const Lens& lens, bool full, const View& Q, const void* Kc, const void* Vc,
                  const int32_t* cu_budget, int64_t capacity, const View& K2, const View& V2, float scale,
                  const View& O, float* lse, void* workspace, hipStream_t stream) {
  AttendParams prm;
  prm.Q = Q;
  prm.K2 = K2;
  prm.V2 = V2;
  prm.O = O;
  prm.lens = lens;
  prm.Kc = reinterpret_cast<const char*>(Kc);
  prm.Vc = reinterpret_cast<const char*>(Vc);
  prm.cu = cu_budget;
  prm.capacity = capacity;
  prm.H = d->H;
  prm.BH = d->B * d->H;
  prm.n_resp = d->n_resp;
  prm.q_per_kv = query_heads_per_kv(d);
  prm.n_q = d->n_resp * prm.q_per_kv;
  prm.full = full ? 1 : 0;
  prm.n_splits = attend_splits(d, full);
  prm.c = scale * kLog2e;
  prm.lse = lse;
  const bool ordered = attend_is_ordered(d, full, capacity);
  prm.ranked = ordered && d->dtype == MASKKV_BF16 && prm.BH <= kRankHeads;
  prm.streamed = attend_is_streamed(d, lens, full);
  prm.order = ordered && !prm.ranked ? reinterpret_cast<const int32_t*>(workspace) : nullptr;
  prm.part_o = nullptr;
  prm.part_ml = nullptr;
  if (prm.n_splits > 1) {
    const size_t rows = (size_t)d->B * d->H * prm.n_splits * prm.n_q;
    prm.part_o = reinterpret_cast<float*>(workspace);
    prm.part_ml = reinterpret_cast<float2*>(reinterpret_cast<char*>(workspace) +
                                            (rows * d->d * sizeof(float) + 255) / 256 * 256);
  }
  if (full ? attend_full_is_narrow(d, lens) : attend_is_narrow(d, full, capacity)) {
    if (d->dtype == MASKKV_BF16) return d->d == 128 ? launch_attend_pairs<128>(prm, stream) : launch_attend_pairs<64>(prm, stream);
    if (attend_is_small(d)) return d->d == 128 ? launch_attend_small<128>(prm, stream) : launch_attend_small<64>(prm, stream);
    return d->d == 128 ? launch_attend_narrow<128>(prm, stream) : launch_attend_narrow<64>(prm, stream);
  }
  if (d->dtype == MASKKV_BF16)
    return d->d == 128 ? launch_attend_t<bf16_t, 128>(prm, d->B, stream) : launch_attend_t<bf16_t, 64>(prm, d->B, stream);
  return d->d == 128 ? launch_attend_t<float, 128>(prm, d->B, stream) : launch_attend_t<float, 64>(prm, d->B, stream);
}

}  // namespace maskkv
