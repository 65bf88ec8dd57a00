// What the attention kernels share.
#pragma once

#include "kernels.hpp"
#include "lds.hpp"

namespace maskkv {

constexpr float kLazyBump = 8.f;  // log2 of the largest probability tolerated before the running reference is raised

constexpr int kRankHeads = 256;   // heads up to which the tiled bf16 kernel's workgroups find the heads' order themselves

struct AttendParams {
  View Q, K2, V2, O;
  Lens lens;
  const char* Kc;
  const char* Vc;
  const int32_t* cu;
  int64_t capacity;
  int H, BH, n_resp, full, n_splits;
  int q_per_kv;  // query heads per key/value head
  int n_q;       // query rows per key/value head = q_per_kv * n_resp
  float c;  // scale * log2(e)
  float* lse;
  int ranked;            // they do (see kRankHeads)
  int streamed;          // V passes by the memory-side cache (see attend_is_streamed)
  const int32_t* order;  // [BH] heads by descending key count (compressed call of the tiled kernel), or null
  float* part_o;     // [BH][n_splits][n_q][D]
  float2* part_ml;   // [BH][n_splits][n_q]
};

// GRID: the kernel uses the size of its grid, which lies behind the parameter.
template <bool GRID>
__device__ __forceinline__ void fetch_attend_arguments() {
  typedef AttendParams A;
  fetch_arguments({MASKKV_VIEW_ARGUMENTS(A, Q), MASKKV_VIEW_ARGUMENTS(A, K2), MASKKV_VIEW_ARGUMENTS(A, V2), MASKKV_VIEW_ARGUMENTS(A, O),
                   MASKKV_ARGUMENT(A, lens), MASKKV_ARGUMENT(A, Kc), MASKKV_ARGUMENT(A, H), (uint32_t)(GRID ? sizeof(A) : offsetof(A, part_o))});
}

// Rows of V (bf16) in LDS as direct transfers leave them: no padding, the 32-byte unit u of a row in slot u ^ v_swizzle(row).  A
// transposing read takes 32 bytes of four rows per 16 lanes and 64 bytes of four rows per 32 lanes, and both sets fall on
// different banks.
template <int D>
__device__ __forceinline__ uint32_t v_swizzle(uint32_t row) {
  return D == 128 ? ((row & 3) << 1 | (row & 3) >> 1) : row & 3;
}
// Where a lane points for keys 4g .. 4g+3 of the A operand of O^T = V^T P^T, head-dim elements 32 db .. (keys 8 on: 8 rows on).
template <int D>
__device__ __forceinline__ uint32_t v_read_offset(uint32_t lane, uint32_t db) {
  const uint32_t i = lane & 15, row = i >> 2;
  return (4 * (lane >> 5) + row) * (2 * D) + (((2 * db + ((lane >> 4) & 1)) ^ v_swizzle<D>(row)) << 5) + (i & 3) * 8;
}

typedef __attribute__((ext_vector_type(4))) short s16x4;

// LDS read of 8 bytes a lane with a transposition inside each group of 16 lanes: lanes 4j .. 4j+3 point at 16 elements of row j,
// lane i receives element i of rows 0 .. 3.
__device__ __forceinline__ u32x2 read_transposed(uint32_t addr, int imm) {
  return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(in_lds<s16x4>(addr, imm)));
}

// attend_tiles.hip: the tiled kernel for bf16.
// Queries per workgroup for `units` heads of n_q query rows.
int attend_tiles_queries(int64_t units, int n_q, bool full);
int launch_attend_tiles(const AttendParams& prm, int d, int queries, hipStream_t stream);

struct KeySpace {
  const char* a_k;  // packed segment base (row 0 of this head), rows contiguous
  const char* a_v;
  int len_a;
  int len_b;
};

}  // namespace maskkv
