// Internal launch interface between the C ABI (api.hip) and the kernel files.
#pragma once

#include "common.hpp"

namespace maskkv {

// How the single sweep's workgroups are dealt out (sweep.hip).  A run: from workgroup `place` on, `side` heads of a sequence side by
// side, `width` workgroups in all, for its heads from `head` on, `times` times.  The runs of a round follow each other and have the
// same number of times.
constexpr int kMaxRuns = 2 * MASKKV_MAX_BATCH;
struct SweepPlan {
  int groups;   // workgroups, or 0: two passes
  int grid;     // of the launch; where there are more groups, each half of a workgroup is one
  int subsets;  // a head's groups of voting rows are dealt to as many sets of workgroups
  int runs;
  int rounds;   // the most chunks of a workgroup
  int parts;    // not 0: no sweep, but a head's voting rows are dealt to so many workgroups that keep all of their keys (rows.hip)
  uint32_t places[kMaxRuns], heads[kMaxRuns], repeats[kMaxRuns];
  __host__ __device__ bool halves() const { return groups > grid; }
  __host__ __device__ int place(int i) const { return places[i] & 0xFFFF; }
  __host__ __device__ int width(int i) const { return places[i] >> 16; }
  __host__ __device__ int head(int i) const { return heads[i] & 0xFFFF; }
  __host__ __device__ int side(int i) const { return heads[i] >> 16; }
  __host__ __device__ int times(int i) const { return repeats[i] & 0xFFFF; }
  __host__ __device__ int sequence(int i) const { return repeats[i] >> 16; }
  __host__ __device__ bool has(int i, int w) const { return w >= place(i) && w < place(i) + width(i); }
  void put(int i, int p, int s, int w, int b, int h) {
    places[i] = (uint32_t)p | (uint32_t)w << 16;
    heads[i] = (uint32_t)h | (uint32_t)s << 16;
    repeats[i] = (uint32_t)b << 16;
  }
  void repeat(int i, int t) { repeats[i] |= (uint32_t)t; }
};

// score.hip.  (Choosing takes 0.4 to 1.5 us of host time and up to 30 for 64 sequences of different lengths: once per call.)
SweepPlan score_sweep_plan(const maskkv_desc* d, const Lens& lens);
size_t score_workspace_bytes(const maskkv_desc* d, const Lens& lens, const SweepPlan& plan);
int launch_score(const maskkv_desc* d, const View& Q, const View& K, const Lens& lens, float scale, float* scores,
                 int64_t score_stride, float* prompt_mass, void* workspace, hipStream_t stream,
                 void* const* events, const SweepPlan& plan, const float* row_lse = nullptr);

// rows.hip: the scores of short fp32 prompts in one pass.  score_rows_parts: column sums per head that it leaves, or 0 where it does not apply.
struct RowsParams {
  View Q, K;
  Lens lens;
  int B, H, n_resp;
  int n_query;      // voting rows per key/value head: q_per_kv query heads of n_qh mask queries each
  int n_qh, q_per_kv;
  float c;          // scale * log2(e)
  float* out;       // [B*H][parts][out_stride]
  int64_t out_stride;
  float* mass;      // [B*H][parts] or null
  int part_keys, parts;  // not 0: keys are dealt out in so many parts of so many keys
  float4* stats;    // [B*H][n_query][parts]
};
struct RowsSplit {
  int groups;            // groups of 16 rows a workgroup of the first kernel: 1 (and 32 keys a workgroup of the second) or 2 (64)
  int part_keys, parts;  // keys a workgroup of the first, and how many of them, or 0
};
// Whether rows and keys are both dealt out, and how.
RowsSplit score_rows_split(const maskkv_desc* d, const Lens& lens);
size_t score_rows_split_bytes(const maskkv_desc* d, const RowsSplit& split);
RowsSplit score_split(const maskkv_desc* d, const Lens& lens, const SweepPlan& plan);  // (as far as the workspace has room for it)
int score_rows_parts(const maskkv_desc* d, const Lens& lens);
int launch_score_rows(const RowsParams& prm, int d, int parts, const RowsSplit& split, hipStream_t stream);

// sweep.hip: the scores in one sweep over the keys
SweepPlan sweep_plan(const maskkv_desc* d, const Lens& lens, int nqg);
size_t sweep_workspace_bytes(const maskkv_desc* d, int nqg, const SweepPlan& plan);
// for tests and measurements: marks the device's sweep as taken age_us ago, as by a call that has not ended (age_us < 0: not taken)
int hold_sweep(int64_t age_us, hipStream_t stream);
int launch_sweep(const maskkv_desc* d, const View& Q, const View& K, const Lens& lens, float scale, float* scores,
                 int64_t score_stride, float* prompt_mass, float* group_sums, int64_t group_stride, int nqg, const SweepPlan& plan,
                 void* area, hipStream_t stream, float** unit_mass);

// select.hip
size_t select_workspace_bytes(const maskkv_desc* d);
int64_t select_max_prompt();
int launch_select(const maskkv_desc* d, const Lens& lens, const float* scores, int64_t score_stride, int window,
                  int mode, const int32_t* budgets, int32_t* idx, int32_t* cu_budget, int64_t capacity,
                  void* workspace, hipStream_t stream);
int launch_head_budgets(const maskkv_desc* d, const float* prompt_mass, int32_t k_l, float alpha, int32_t* budgets,
                        hipStream_t stream);

// compact.hip
int launch_compact(const maskkv_desc* d, const Lens& lens, const View& K, const View& V, const int32_t* idx, const int32_t* cu_budget,
                   int64_t capacity, void* Kc, void* Vc, hipStream_t stream);

// attend.hip
size_t attend_workspace_bytes(const maskkv_desc* d, bool full);
int launch_attend(const maskkv_desc* d, const Lens& lens, bool full, const View& Q, const void* Kc, const void* Vc,
                  const int32_t* cu_budget, int64_t capacity, const View& K2, const View& V2, float scale,
                  const View& O, float* lse, void* workspace, hipStream_t stream);

// layer.hip
size_t layer_importance_workspace_bytes();
int launch_layer_importance(const void* h_in, const void* h_out, int64_t n, int hidden, int dtype, int64_t row_bytes,
                            float* importance, void* workspace, hipStream_t stream);
int launch_value_shift(const void* v_now, const void* v_prev, int64_t n, int width, int dtype, int64_t row_bytes,
                       float delta, float* cos, int32_t* refresh, int32_t* count, hipStream_t stream);

// api.hip: the body of maskkv_score.  events: null, or four hipEvent_t (each may be null) recorded on the stream
// before the first kernel, before the merge and before pass 2 (or both behind the sweep kernel), and after the last;
// measurement harnesses link against this to time the stages of one call (the C entry point always passes null).
int score_entry(const maskkv_desc* desc, const maskkv_tensor* Q_mask, const maskkv_tensor* K_full, float scale,
                float* scores, int64_t score_stride, float* prompt_mass, void* workspace, size_t workspace_bytes,
                void* stream, void* const* events);
// The plan that it makes for a description, and whether it deals out rows and keys instead.
int score_plan(const maskkv_desc* desc, SweepPlan* plan, RowsSplit* split);

}  // namespace maskkv
