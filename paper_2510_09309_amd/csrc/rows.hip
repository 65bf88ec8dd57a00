// Mask-Voting scores of short fp32 prompts in one pass (see score.hip for the definitions and the two-pass form).
//
// A workgroup of eight waves takes 16 voting rows of a head over all of its keys: logits and exponentials of 16 rows x 3072 keys
// fit the registers (96 per lane), so rows are normalised without a second pass and without another workgroup's sums.  Its
// column sums are the scores themselves, or parts of them that a last small kernel adds in a fixed order.
//
// Rows are on the MFMA's row axis (16x16: element i of a lane is row 4 * (lane / 16) + i, key lane % 16); the fragments of rows and
// keys are 16 bytes of a row per lane, straight from global memory, 8 or 16 of keys in flight.  Wave w has every eighth tile of 16 keys.
//
// What bounds it: latency (launch, first fragments, two exchanges of the waves' maxima and sums, the last kernel: 9 us of a call),
// then the fp32 MFMAs of as many workgroups as there are groups of rows.  us a call, three kernels of two passes before: 4 heads x 64
// rows x 576 keys of dimension 64 20.5 -> 13.4, 4 x 32 x 332 of 128 33.3 -> 14, 12 x 128 x 2628 of 128 67.6 -> 52.6.  In bf16 the
// same kernel takes 11 us for the smallest prompts, the sweep 12.5, but 37 against 15 for 12 x 128 x 2628: not kept.
#include "kernels.hpp"

namespace maskkv {

namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int kWaves = 8;
constexpr int kThreads = 64 * kWaves;
constexpr int kRowsWG = 16;
constexpr int kTile = 16;      // keys
constexpr int kMaxTiles = 24;  // of a wave (32: registers are spilled)
constexpr int kMaxKeys = kMaxTiles * kWaves * kTile;

__device__ __forceinline__ void mfma16(const u32x4& a, const u32x4& b, f32x4& acc) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const uint32_t ua = a[q], ub = b[q];
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(as_f32(ua), as_f32(ub), acc, 0, 0, 0);
  }
}

template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, false));
}
__device__ __forceinline__ float sum16(float v) {  // over 16 lanes, in each of them
  v += dpp<0xB1>(v);
  v += dpp<0x4E>(v);
  v += dpp<0x141>(v);
  return v + dpp<0x140>(v);
}
__device__ __forceinline__ float max16(float v) {
  v = fmaxf(v, dpp<0xB1>(v));
  v = fmaxf(v, dpp<0x4E>(v));
  v = fmaxf(v, dpp<0x141>(v));
  return fmaxf(v, dpp<0x140>(v));
}
__device__ __forceinline__ float sum_quarters(float v) {  // over the lanes of the same number modulo 16
  const auto a = __builtin_amdgcn_permlane16_swap(as_u32(v), as_u32(v), false, false);
  const unsigned a0 = a[0], a1 = a[1];
  v = as_f32(a0) + as_f32(a1);
  const auto b = __builtin_amdgcn_permlane32_swap(as_u32(v), as_u32(v), false, false);
  const unsigned b0 = b[0], b1 = b[1];
  return as_f32(b0) + as_f32(b1);
}

// NT: tiles of a wave.  MANY: a workgroup has more than 16 rows, which it takes one after the other.
template <int D, int NT, bool MANY>
__global__ __launch_bounds__(kThreads, 2) void score_rows_kernel(const RowsParams prm) {
  constexpr int S = D * 4 / 64;                                // fragments of a row
  constexpr int kInFlight = D * NT > 128 * 16 ? 8 : 16;        // fragments of keys (as the registers allow)
  __shared__ float wave_max[kWaves][kRowsWG];
  __shared__ float2 wave_sum[kWaves][kRowsWG];  // over the prompt's keys and the response span's
  const int lane = threadIdx.x & 63, n = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int b = blockIdx.z, h = blockIdx.y, bh = b * prm.H + h;
  const int P = prm.lens.P[b], N = P + prm.n_resp;
  const char* keys = prm.K.row(b, h, 0);
  double mass = 0.;  // (in fp32 the groups' sums, one after the other, would lose more than the two passes' tree does)
  float col[NT];
  if (MANY)
#pragma unroll
    for (int t = 0; t < NT; ++t) col[t] = 0.f;

  const int groups = (prm.n_query + kRowsWG - 1) / kRowsWG;
  const int first = groups * (int)blockIdx.x / (int)gridDim.x, past = groups * ((int)blockIdx.x + 1) / (int)gridDim.x;
  for (int rg = first; rg < (MANY ? past : first + 1); ++rg) {
    const int q0 = rg * kRowsWG;
    u32x4 qf[S];
    const char* qrow = prm.Q.group_row(b, h, prm.q_per_kv, prm.n_qh, min(q0 + n, prm.n_query - 1)) + g * 16;
#pragma unroll
    for (int s = 0; s < S; ++s) qf[s] = *reinterpret_cast<const u32x4*>(qrow + s * 64);
    f32x4 p[NT];
    u32x4 kf[kInFlight];
    auto load = [&](int f) {  // fragment f % S of tile f / S (tiles past the last key re-read it)
      const int key = min((f / S * kWaves + wave) * kTile + n, N - 1);
      kf[f % kInFlight] = *reinterpret_cast<const u32x4*>(keys + (int64_t)key * prm.K.stride_t + (f % S * 64 + g * 16));
    };
#pragma unroll
    for (int f = 0; f < min(kInFlight, NT * S); ++f) load(f);
#pragma unroll
    for (int f = 0; f < NT * S; ++f) {
      if (f % S == 0) p[f / S] = f32x4{};
      mfma16(qf[f % S], kf[f % kInFlight], p[f / S]);
      if (f + kInFlight < NT * S) load(f + kInFlight);
      __builtin_amdgcn_sched_barrier(0);
    }
    // ---- the rows' maxima, in base-2 logits
    float top[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) top[i] = kNegBig;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const bool there = (t * kWaves + wave) * kTile + n < N;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        p[t][i] = there ? p[t][i] * prm.c : -INFINITY;
        top[i] = fmaxf(top[i], p[t][i]);
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      top[i] = max16(top[i]);
      if (n == 0) wave_max[wave][4 * g + i] = top[i];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int w = 0; w < kWaves; ++w) top[i] = fmaxf(top[i], wave_max[w][4 * g + i]);
    // ---- exponentials and the rows' sums
    float lp[4] = {}, lr[4] = {};
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const bool prompt = (t * kWaves + wave) * kTile + n < P;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float e = fast_exp2(p[t][i] - top[i]);
        p[t][i] = e;
        lp[i] += prompt ? e : 0.f;
        lr[i] += prompt ? 0.f : e;
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      lp[i] = sum16(lp[i]);
      lr[i] = sum16(lr[i]);
      if (n == 0) wave_sum[wave][4 * g + i] = make_float2(lp[i], lr[i]);
    }
    __syncthreads();
    float w[4], share = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float sp = 0.f, sr = 0.f;
#pragma unroll
      for (int v = 0; v < kWaves; ++v) {
        const float2 x = wave_sum[v][4 * g + i];
        sp += x.x;
        sr += x.y;
      }
      w[i] = q0 + 4 * g + i < prm.n_query ? 1.f / (sp + sr) : 0.f;
      share += sp * w[i];
    }
    mass += share;
    // ---- column sums
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const float v = (p[t][0] * w[0] + p[t][1] * w[1]) + (p[t][2] * w[2] + p[t][3] * w[3]);
      col[t] = MANY ? col[t] + v : v;
    }
  }
  const int64_t part = (int64_t)bh * gridDim.x + blockIdx.x;
  float* out = prm.out + part * prm.out_stride;
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int key = (t * kWaves + wave) * kTile + n;
    const float v = sum_quarters(col[t]);
    if (lane < 16 && key < P) out[key] = v;
  }
  const float all = sum_quarters((float)mass);  // (every lane of a quarter has the same)
  if (threadIdx.x == 0 && prm.mass) prm.mass[part] = all;
}

template <int D, int NT>
int launch(const RowsParams& prm, const dim3& grid, hipStream_t stream) {
  if ((int)grid.x * kRowsWG >= prm.n_query)
    hipLaunchKernelGGL((score_rows_kernel<D, NT, false>), grid, dim3(kThreads), 0, stream, prm);
  else
    hipLaunchKernelGGL((score_rows_kernel<D, NT, true>), grid, dim3(kThreads), 0, stream, prm);
  return check_launch("score (rows)");
}

template <int D>
int launch(const RowsParams& prm, const dim3& grid, int tiles, hipStream_t stream) {
  if (tiles <= 3) return launch<D, 3>(prm, grid, stream);
  if (tiles <= 5) return launch<D, 5>(prm, grid, stream);
  if (tiles <= 8) return launch<D, 8>(prm, grid, stream);
  if (tiles <= 12) return launch<D, 12>(prm, grid, stream);
  if (tiles <= 16) return launch<D, 16>(prm, grid, stream);
  return launch<D, kMaxTiles>(prm, grid, stream);
}

}  // namespace

// Microseconds of a call (measured over 1 ... 256 heads, 16 ... 896 rows, 300 ... 2900 keys).  This kernel: 9 and, for every tile
// of a wave and round of workgroups, 2.4 (head_dim 64: 1.2); the two passes: 33 (20) and 0.068 (0.027) per 64 keys x 256 rows.  They are
// the faster way for few rows over long prompts (1 head x 16 rows x 2916 keys: 35 against 49) and for large batches.
int score_rows_parts(const maskkv_desc* d, const Lens& lens) {
  if (d->dtype != MASKKV_F32 || d->H > 65535) return 0;
  const int64_t rows = (int64_t)d->n_query * query_heads_per_kv(d), bh = (int64_t)d->B * d->H;
  const int64_t groups = (rows + kRowsWG - 1) / kRowsWG;
  int most = 0;
  int64_t blocks = 0;
  for (int b = 0; b < d->B; ++b) {
    most = max(most, lens.P[b]);
    blocks += (lens.P[b] + 63) / 64 + (d->n_resp + 63) / 64;
  }
  if (most == 0 || most + d->n_resp > kMaxKeys) return 0;
  blocks *= d->H * ((rows + 255) / 256);
  const int tiles = (most + d->n_resp + kWaves * kTile - 1) / (kWaves * kTile);
  const bool wide = d->d == 128;
  const double here = 9.0 + (wide ? 2.4 : 1.2) * tiles * fmax(1.0, (double)(bh * groups) / 256);
  if (here > (wide ? 33.0 : 20.0) + (wide ? 0.068 : 0.027) * (double)blocks) return 0;
  return (int)min(groups, max((int64_t)1, 512 / bh));
}

int launch_score_rows(const RowsParams& prm, int d, int parts, hipStream_t stream) {
  int most = 0;
  for (int b = 0; b < prm.B; ++b) most = max(most, prm.lens.P[b]);
  const int tiles = (most + prm.n_resp + kWaves * kTile - 1) / (kWaves * kTile);
  const dim3 grid(parts, prm.H, prm.B);
  return d == 128 ? launch<128>(prm, grid, tiles, stream) : launch<64>(prm, grid, tiles, stream);
}

}  // namespace maskkv
