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
// then the fp32 MFMAs of as many workgroups as there are groups of rows.  us a call, three kernels of two passes before: 12 heads x 128
// rows x 2628 keys of dimension 128 67.6 -> 52.6.  In bf16 the same kernel takes 37 where the sweep takes 15: not kept.
//
// Where that leaves most of the chip idle, both rows and keys are dealt out (score_rows_split) and the logits formed twice: 4 heads x 64 rows
// x 576 keys of dimension 64, whose 16 workgroups spend 6.7 of 8.4 us on their products, 13.0 -> 10.1 us, 4 x 36 x 580 of 128 17.5 ->
// 11.8.  What bounds that: two kernels of 2.5 us and their launches, then fragments straight from memory, which each wave needs for itself.
#include "kernels.hpp"

namespace maskkv {

namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int kWaves = 8;
constexpr int kThreads = 64 * kWaves;
constexpr int kRowsWG = 16;
constexpr int kStatWaves = 4;
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

__device__ __forceinline__ void fetch_rows_arguments() {
  typedef RowsParams R;
  fetch_arguments({MASKKV_VIEW_ARGUMENTS(R, Q), MASKKV_VIEW_ARGUMENTS(R, K), MASKKV_ARGUMENT(R, lens), MASKKV_ARGUMENT(R, B), MASKKV_ARGUMENT(R, out),
                   MASKKV_ARGUMENT(R, stats)});
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
  fetch_rows_arguments();
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

// ---- few workgroups' worth of rows: the keys are dealt out as well, and the logits formed twice.
//
// A workgroup of rows_stats_kernel has 16 * RG rows and prm.part_keys keys of a head (each of its waves every fourth 16 of them) and leaves each
// row's maximum and its sums over prompt and response keys; one of rows_columns_kernel has 16 * NT keys, takes the rows' normalisers from
// all of these and adds its columns over all rows.

template <int D, int RG>
__global__ __launch_bounds__(64 * kStatWaves) void rows_stats_kernel(const RowsParams prm) {
  constexpr int S = D * 4 / 64;
  __shared__ float4 of_wave[kStatWaves][RG * kRowsWG];
  fetch_rows_arguments();
  const int lane = threadIdx.x & 63, n = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int bh = blockIdx.z, b = prm.B == 1 ? 0 : bh / prm.H, h = bh - b * prm.H;
  const int P = prm.lens.P[b], N = P + prm.n_resp, q0 = (int)blockIdx.y * (RG * kRowsWG);
  const int past = min(N, ((int)blockIdx.x + 1) * prm.part_keys);
  const char* keys = prm.K.row(b, h, 0) + g * 16;
  u32x4 qf[RG][S], kf[S];
  auto load_k = [&](int key0) {
    const char* krow = keys + (int64_t)min(key0 + n, N - 1) * prm.K.stride_t;
#pragma unroll
    for (int s = 0; s < S; ++s) kf[s] = *reinterpret_cast<const u32x4*>(krow + s * 64);
  };
  int key0 = (int)blockIdx.x * prm.part_keys + wave * kTile;  // this wave's tile
  load_k(key0);
#pragma unroll
  for (int r = 0; r < RG; ++r) {
    const char* qrow = prm.Q.group_row(b, h, prm.q_per_kv, prm.n_qh, min(q0 + r * kRowsWG + n, prm.n_query - 1)) + g * 16;
#pragma unroll
    for (int s = 0; s < S; ++s) qf[r][s] = *reinterpret_cast<const u32x4*>(qrow + s * 64);
  }
  __builtin_amdgcn_sched_barrier(0);  // (all of them asked for before the first product)
  // each lane has the maximum and the sums of the keys that it sees
  float top[RG][4], lp[RG][4], lr[RG][4];
#pragma unroll
  for (int r = 0; r < RG; ++r)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      top[r][i] = kNegBig;
      lp[r][i] = lr[r][i] = 0.f;
    }
  for (; key0 < past; key0 += kStatWaves * kTile) {
    f32x4 a[RG];
#pragma unroll
    for (int r = 0; r < RG; ++r) a[r] = f32x4{};
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
      for (int r = 0; r < RG; ++r) mfma16(qf[r][s], kf[s], a[r]);
    __builtin_amdgcn_sched_barrier(0);
    if (key0 + kStatWaves * kTile < past) load_k(key0 + kStatWaves * kTile);
    __builtin_amdgcn_sched_barrier(0);
    const bool there = key0 + n < N, prompt = key0 + n < P;
#pragma unroll
    for (int r = 0; r < RG; ++r)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float m = there ? fmaxf(top[r][i], a[r][i] * prm.c) : top[r][i];
        const float e = there ? fast_exp2(fmaf(a[r][i], prm.c, -m)) : 0.f, keep = fast_exp2(top[r][i] - m);
        lp[r][i] = fmaf(lp[r][i], keep, prompt ? e : 0.f);
        lr[r][i] = fmaf(lr[r][i], keep, prompt ? 0.f : e);
        top[r][i] = m;
      }
  }
#pragma unroll
  for (int r = 0; r < RG; ++r)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float m = max16(top[r][i]), f = fast_exp2(top[r][i] - m);
      const float p = sum16(lp[r][i] * f), q = sum16(lr[r][i] * f);
      if (n == 0) of_wave[wave][r * kRowsWG + 4 * g + i] = make_float4(m, p, q, 0.f);
    }
  __syncthreads();
  if ((int)threadIdx.x < RG * kRowsWG && q0 + (int)threadIdx.x < prm.n_query) {
    float4 v[kStatWaves];
    float m = kNegBig, p = 0.f, r = 0.f;
#pragma unroll
    for (int w = 0; w < kStatWaves; ++w) {
      v[w] = of_wave[w][threadIdx.x];
      m = fmaxf(m, v[w].x);
    }
#pragma unroll
    for (int w = 0; w < kStatWaves; ++w) {
      const float f = fast_exp2(v[w].x - m);
      p += v[w].y * f;
      r += v[w].z * f;
    }
    prm.stats[((int64_t)bh * prm.n_query + q0 + threadIdx.x) * gridDim.x + blockIdx.x] = make_float4(m, p, r, 0.f);
  }
}

template <int D, int NT>
__global__ __launch_bounds__(kThreads) void rows_columns_kernel(const RowsParams prm) {
  constexpr int S = D * 4 / 64;
  __shared__ float of_wave[kWaves][NT * kTile];
  __shared__ double mass_of_wave[kWaves];
  fetch_rows_arguments();
  const int lane = threadIdx.x & 63, n = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int bh = blockIdx.y, b = prm.B == 1 ? 0 : bh / prm.H, h = bh - b * prm.H;
  const int P = prm.lens.P[b], key0 = (int)blockIdx.x * NT * kTile;
  if (key0 >= P && blockIdx.x > 0) return;  // (the first one has the mass, also that of an empty prompt)
  const int groups = (prm.n_query + kRowsWG - 1) / kRowsWG, parts = (P + prm.n_resp + prm.part_keys - 1) / prm.part_keys;
  u32x4 kf[NT][S];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const char* krow = prm.K.row(b, h, 0) + (int64_t)min(key0 + t * kTile + n, P + prm.n_resp - 1) * prm.K.stride_t + g * 16;
#pragma unroll
    for (int s = 0; s < S; ++s) kf[t][s] = *reinterpret_cast<const u32x4*>(krow + s * 64);
  }
  float col[NT] = {};
  double mass = 0.;
  for (int rg = wave; rg < groups; rg += kWaves) {
    const char* qrow = prm.Q.group_row(b, h, prm.q_per_kv, prm.n_qh, min(rg * kRowsWG + n, prm.n_query - 1)) + g * 16;
    u32x4 qf[S];
#pragma unroll
    for (int s = 0; s < S; ++s) qf[s] = *reinterpret_cast<const u32x4*>(qrow + s * 64);
    // lane n of a quarter has every sixteenth part of the quarter's rows
    const float4* st[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) st[i] = prm.stats + ((int64_t)bh * prm.n_query + min(rg * kRowsWG + 4 * g + i, prm.n_query - 1)) * prm.parts;
    float m[4], lp[4], lr[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      m[i] = kNegBig;
      lp[i] = lr[i] = 0.f;
    }
    for (int p0 = 0; p0 < parts; p0 += 16) {
      float4 v[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = st[i][min(p0 + n, parts - 1)];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float x = p0 + n < parts ? v[i].x : kNegBig, top = fmaxf(m[i], x);
        const float keep = fast_exp2(m[i] - top), add = p0 + n < parts ? fast_exp2(x - top) : 0.f;
        lp[i] = fmaf(v[i].y, add, lp[i] * keep);
        lr[i] = fmaf(v[i].z, add, lr[i] * keep);
        m[i] = top;
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    f32x4 a[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) a[t] = f32x4{};
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
      for (int t = 0; t < NT; ++t) mfma16(qf[s], kf[t][s], a[t]);
    float w[4], share = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float top = max16(m[i]), f = fast_exp2(m[i] - top);
      const float sp = sum16(lp[i] * f), sr = sum16(lr[i] * f);
      m[i] = top;
      w[i] = rg * kRowsWG + 4 * g + i < prm.n_query ? 1.f / (sp + sr) : 0.f;
      share += sp * w[i];
    }
    mass += share;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      float e[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) e[i] = fast_exp2(fmaf(a[t][i], prm.c, -m[i]));
      col[t] += (e[0] * w[0] + e[1] * w[1]) + (e[2] * w[2] + e[3] * w[3]);
    }
  }
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const float v = sum_quarters(col[t]);
    if (lane < kTile) of_wave[wave][t * kTile + lane] = v;
  }
  if (blockIdx.x == 0) {  // (every lane of a quarter has the same)
    mass += __shfl_xor(mass, 16, 64);
    mass += __shfl_xor(mass, 32, 64);
    if (lane == 0) mass_of_wave[wave] = mass;
  }
  __syncthreads();
  if ((int)threadIdx.x < NT * kTile && key0 + (int)threadIdx.x < P) {
    float v = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) v += of_wave[w][threadIdx.x];
    prm.out[(int64_t)bh * prm.out_stride + key0 + threadIdx.x] = v;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0 && prm.mass) {
    double m = 0.;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) m += mass_of_wave[w];
    prm.mass[bh] = (float)m;
  }
}

template <int D, int RG, int NT>
int launch_split(const RowsParams& prm, int most, hipStream_t stream) {
  const dim3 first(prm.parts, (prm.n_query + RG * kRowsWG - 1) / (RG * kRowsWG), prm.B * prm.H);
  hipLaunchKernelGGL((rows_stats_kernel<D, RG>), first, dim3(64 * kStatWaves), 0, stream, prm);
  if (int e = check_launch("score (rows' sums)")) return e;
  const dim3 grid(max(1, (most + NT * kTile - 1) / (NT * kTile)), prm.B * prm.H);
  hipLaunchKernelGGL((rows_columns_kernel<D, NT>), grid, dim3(kThreads), 0, stream, prm);
  return check_launch("score (columns)");
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

// Microseconds of a call (measured over 1 ... 256 heads, 16 ... 896 rows, 300 ... 2900 keys).  The one pass: 9 and, for every tile
// of a wave and round of workgroups, 2.4 (head_dim 64: 1.2); the two passes: 33 (20) and 0.068 (0.027) per 64 keys x 256 rows.  They are
// the faster way for few rows over long prompts (1 head x 16 rows x 2916 keys: 35 against 49) and for large batches.
double one_pass_us(const maskkv_desc* d, const Lens& lens) {
  const int64_t groups = ((int64_t)d->n_query * query_heads_per_kv(d) + kRowsWG - 1) / kRowsWG, bh = (int64_t)d->B * d->H;
  int most = 0;
  for (int b = 0; b < d->B; ++b) most = max(most, lens.P[b]);
  const int tiles = (most + d->n_resp + kWaves * kTile - 1) / (kWaves * kTile);
  return 9.0 + (d->d == 128 ? 2.4 : 1.2) * tiles * fmax(1.0, (double)(bh * groups) / 256);
}

double two_passes_us(const maskkv_desc* d, const Lens& lens) {
  int64_t blocks = 0;
  for (int b = 0; b < d->B; ++b) blocks += (lens.P[b] + 63) / 64 + (d->n_resp + 63) / 64;
  blocks *= d->H * (((int64_t)d->n_query * query_heads_per_kv(d) + 255) / 256);
  return (d->d == 128 ? 33.0 : 20.0) + (d->d == 128 ? 0.068 : 0.027) * (double)blocks;
}

}  // namespace

int score_rows_parts(const maskkv_desc* d, const Lens& lens) {
  if (d->dtype != MASKKV_F32 || d->H > 65535) return 0;
  const int64_t rows = (int64_t)d->n_query * query_heads_per_kv(d), bh = (int64_t)d->B * d->H;
  const int64_t groups = (rows + kRowsWG - 1) / kRowsWG;
  int most = 0;
  for (int b = 0; b < d->B; ++b) most = max(most, lens.P[b]);
  if (most == 0 || most + d->n_resp > kMaxKeys) return 0;
  if (one_pass_us(d, lens) > two_passes_us(d, lens)) return 0;
  return (int)min(groups, max((int64_t)1, 512 / bh));
}

// Microseconds of a call: the one pass and the two passes as above; split, with P products of 16 rows and 16 keys, 9.2 + 0.0022 P (head_dim
// 128: 10.5 + 0.0041 P) or, with more for a wave to do, 13.3 + 0.0012 P (17.5 + 0.0024 P).  Measured over 1 ... 96 heads, 16 ... 896 rows, 300 ... 2700 keys,
// each way (the better of the two others / split, the former form / split, the latter): head_dim 64, 4 heads x 64 rows x 576 keys 13.0 / 10.1 /
// 14.7, 4 x 32 x 332 10.5 / 9.4 / 13.5, 8 x 100 x 1300 20.7 / 18.7 / 16.6, 4 x 128 x 2628 24.0 / 21.9 / 17.2, 12 x 256 x 1564 27.1 / 45.3 / 38.7;
// 128, 4 x 36 x 580 17.5 / 11.8 / 18.8, 4 x 32 x 2532 37.3 / 17.3 / 18.1, 4 x 428 x 1515 37.2 / 45.4 / 44.7, 12 x 128 x 2628 52.3 / 75.8 / 52.0.
RowsSplit score_rows_split(const maskkv_desc* d, const Lens& lens) {
  const int64_t rows = (int64_t)d->n_query * query_heads_per_kv(d), bh = (int64_t)d->B * d->H;
  const int64_t groups = (rows + kRowsWG - 1) / kRowsWG;
  int most = 0;
  int64_t products = 0;
  for (int b = 0; b < d->B; ++b) {
    most = max(most, lens.P[b]);
    products += groups * d->H * ((lens.P[b] + d->n_resp + kTile - 1) / kTile);
  }
  if (d->dtype != MASKKV_F32 || most == 0 || most + d->n_resp > kMaxKeys || bh > 65535 || groups > 65535) return RowsSplit{};
  const bool wide = d->d == 128;
  const double few = (wide ? 10.5 : 9.2) + (wide ? 0.0041 : 0.0022) * (double)products;
  // (and, beyond a round of the second kernel's workgroups, 5 for a round that is begun: 12 x 77 x 1478 keys, head_dim 64, 21.2, x 1377 16.1)
  const double rounds = (double)(bh * ((most + 63) / 64)) / 256;
  const double many = (wide ? 17.5 : 13.3) + (wide ? 0.0024 : 0.0012) * (double)products + (rounds > 1 ? 5.0 * (ceil(rounds) - rounds) : 0.0);
  const double groups_sum = rows > 256 ? 5.0 : 0.0;  // the two passes' last kernel
  if (fmin(few, many) > 0.9 * fmin(one_pass_us(d, lens), two_passes_us(d, lens) + groups_sum)) return RowsSplit{};
  RowsSplit s = few < many ? RowsSplit{1, most + d->n_resp > 1024 ? 128 : 64, 0} : RowsSplit{2, 256, 0};
  s.parts = (most + d->n_resp + s.part_keys - 1) / s.part_keys;
  return s;
}

size_t score_rows_split_bytes(const maskkv_desc* d, const RowsSplit& s) {
  return (size_t)d->B * d->H * d->n_query * query_heads_per_kv(d) * s.parts * sizeof(float4);
}

int launch_score_rows(const RowsParams& prm, int d, int parts, const RowsSplit& split, hipStream_t stream) {
  int most = 0;
  for (int b = 0; b < prm.B; ++b) most = max(most, prm.lens.P[b]);
  const int tiles = (most + prm.n_resp + kWaves * kTile - 1) / (kWaves * kTile);
  if (split.parts) {
    if (split.groups == 1) return d == 128 ? launch_split<128, 1, 2>(prm, most, stream) : launch_split<64, 1, 2>(prm, most, stream);
    return d == 128 ? launch_split<128, 2, 4>(prm, most, stream) : launch_split<64, 2, 4>(prm, most, stream);
  }
  const dim3 grid(parts, prm.H, prm.B);
  return d == 128 ? launch<128>(prm, grid, tiles, stream) : launch<64>(prm, grid, tiles, stream);
}

}  // namespace maskkv
