// What the attention kernels share.
#pragma once

#include "kernels.hpp"

namespace maskkv {

constexpr float kLazyBump = 8.f;  // log2 of the largest probability tolerated before the running reference is raised

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
  const int32_t* order;  // [BH] heads by descending key count (compressed call of the tiled kernel), or null
  float* part_o;     // [BH][n_splits][n_q][D]
  float2* part_ml;   // [BH][n_splits][n_q]
};

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
