// Internal declarations shared by the HIP sources of libdare (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "attn_route.h"
#include "dare.h"
#include "dare_kernels.h"
#include "gemm_route.h"

namespace dare {

typedef __bf16 bf16_t;
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// One of n workgroups arrives at *count (device scope, relaxed): true for the last.  The counter wraps to 0
// in the same operation, so calls that overlap against the rules (and then compute what they may) leave it
// at 0 as well once all of their workgroups have arrived, and the next call finds it so.
__device__ __forceinline__ bool arrive_last(unsigned* count, int n) {
  return atomicInc(count, (unsigned)n - 1) == (unsigned)n - 1;
}

constexpr int kWave = 64;

// ---- launchers (defined one per .hip file); all return a hipError_t ----------

struct GemmArgs {
  const void* a;      // [*, lda]
  int lda;
  const void* wt;     // [n, k] packed weight
  int n, k;
  int m_max;          // launch bound on the row count
  const int32_t* idx; // optional row ids (gather of A rows = scatter of C rows)
  const int32_t* m_dev; // optional device row count
  void* c[3];         // output column segments
  int ldc;
  int seg_n;
  float* c32;         // optional fp32 copy of columns [0, c32_cols)
  int c32_cols;
  int k_parts;        // > 1: only c32 is written, as k_parts slabs of partial sums
  long c32_part_stride;
  // rotary embedding of output columns [0, rope_cols) (fp32 table [pos][head_dim/2]
  // of (cos, sin) pairs; position of a row = token id % rope_seq); nullptr = none
  const float* rope;
  int rope_cols, rope_dh, rope_seq;
  // 1: the output columns are (gate, up) pairs of a SwiGLU feed-forward (weight rows
  // interleaved gate_0, up_0, gate_1, ...): column pair (2j, 2j+1) gives one output
  // silu(gate_j) * up_j at column j of c[0] (bf16 path, one segment, no c32)
  int swiglu_pairs;
  // Row list derived inside the kernel (instead of idx and m_dev; bf16: the device-count kernel): the
  // rows are the tokens whose byte in sel_mask [sel_batch * sel_seq] is 0, in
  // ascending order.  The first workgroup also writes what a compaction kernel would:
  // sel_idx_out (and optionally sel_idx_out2) [tokens], sel_off_out [sel_batch + 1],
  // optionally sel_count_out [sel_batch].  At most kSelMaxTokens (fp32: kSelMaxTokensF32)
  // tokens.
  const uint8_t* sel_mask;
  int sel_batch, sel_seq;
  int32_t* sel_idx_out;
  int32_t* sel_idx_out2;
  int32_t* sel_off_out;
  int32_t* sel_count_out;
  // optional workspace for tiles whose k is cut in two (bf16, row count known on the host).  Not for
  // projections with c32, whose sums every mode has to form in one order (the query of an unchanged
  // token then scores exactly 0):
  // gemm_split_tiles_bytes() bytes (the sums of both halves of every tile) and kSplitTiles counters that
  // are 0 before the first launch and that every launch leaves even; one launch at a time
  float* split_tiles;
  int* split_count;
  // > 0 (bf16, a multiple of 64, k of 192 or more): columns [0, part_n) only for the rows part_idx [*part_m_dev] (token ids,
  // as in idx), the others for all rows (idx, m_max); no c32
  int part_n;
  const int32_t* part_idx;
  const int32_t* part_m_dev;
};
constexpr int kSelMaxTokens = 2048, kSelMaxTokensF32 = 1024;
constexpr size_t gemm_split_tiles_bytes() { return (size_t)kSplitTiles * 2 * kPpRows * 128 * sizeof(float); }

// Rotation of the channel pairs (v0, v1) and (v2, v3) by the table's (cos, sin) pairs of both
__device__ __forceinline__ void rope_rotate4(const f32x4 cs, float& v0, float& v1, float& v2, float& v3) {
  const float a0 = v0 * cs[0] - v1 * cs[1], a1 = v0 * cs[1] + v1 * cs[0];
  const float a2 = v2 * cs[2] - v3 * cs[3], a3 = v2 * cs[3] + v3 * cs[2];
  v0 = a0;
  v1 = a1;
  v2 = a2;
  v3 = a3;
}

// Drift score of one token from the sums <q, p>, |q|^2, |p|^2 (Sec. 3.1 eq. 1)
__device__ __forceinline__ float drift_score(float dot, float nq, float np) {
  return 1.0f - dot / fmaxf(sqrtf(nq * np), 1e-30f);
}
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Scored query columns of the listed rows and what follows from them in one launch: drift score,
// reuse decision, score-cache update (bf16; width 64 or 128).
struct ScoreProjArgs {
  const void* a;         // [*, k] hidden states
  const void* wt;        // [width, k] packed weight of the scored columns
  int k, width;
  int k_ranges;          // 1, 2, 4 or 8, dividing k / 64: the sum over k is that of this many ranges
  int m;                 // rows
  const int32_t* idx;    // their token ids, or nullptr: 0 .. m-1
  float* q_prev;         // [*, width] score cache
  float threshold;
  int force_refresh;
  float* scores;         // [*] or nullptr
  uint8_t* mask;         // [*]
  int batch, seq, prefix;  // tokens [0, prefix) of every sequence: mask 1, score 0, nothing else
  // workspace for row tiles whose k is cut over workgroups: fp32 sums, and counters that are 0
  // before the launch and that the launch leaves at 0; nullptr = one workgroup per row tile
  float* sums;
  size_t sums_elems;
  unsigned* count;       // [kScoreTiles]
};
constexpr int kScoreTiles = 256;
hipError_t launch_score_proj(const ScoreProjArgs& g, hipStream_t s);

hipError_t launch_gemm_bf16(const GemmArgs& g, hipStream_t s);
hipError_t launch_gemm_f32(const GemmArgs& g, hipStream_t s);

// Workspace for query blocks whose keys are cut over workgroups (bf16, refreshed rows):
// attn_parts_elems() floats and kAttnParts counters that are 0 before the first launch and
// that every launch leaves at 0; one launch at a time.  Null pointers: keys are never cut.
struct AttnParts {
  float* out;
  unsigned* count;
};

struct AttnArgs {
  const void* q;
  const void* k;
  const void* v;
  void* out;
  int batch, seq, n_heads, head_dim;
  const int32_t* idx;      // optional selected rows
  const int32_t* sel_off;  // [batch+1] when idx != nullptr
  bool many_rows;          // the listed rows are most of each sequence (a frozen prefix), not a few
  int active;              // then: how many of each sequence
  AttnParts parts;
};
constexpr int kAttnParts = 256;  // parts of a launch, at most: one per CU
constexpr size_t attn_parts_elems(int head_dim) { return (size_t)kAttnParts * 64 * 2 * (head_dim / 2 + 2); }
hipError_t launch_attn_bf16(const AttnArgs& a, hipStream_t s);
hipError_t launch_attn_f32(const AttnArgs& a, hipStream_t s);

hipError_t launch_pack_weight(int dtype, const void* w, int rows_k, int cols_n, void* wt,
                              int ldwt, hipStream_t s);
hipError_t launch_score(const float* q_new, int ld_new, int width, int n_parts, long part_stride,
                        float* q_prev, int n_tokens, float threshold, int force_refresh, float* scores, float* scores2,
                        uint8_t* mask, int seq, int prefix, hipStream_t s);
hipError_t launch_compact(const uint8_t* mask, int batch, int seq, int32_t* sel_idx,
                          int32_t* sel_idx2, int32_t* sel_count, int32_t* sel_count2,
                          int32_t* sel_off, hipStream_t s);
hipError_t launch_quantile_mask(const float* scores, int batch, int stride, int first, int seq, int rank,
                                int force_refresh, float* tau_out, uint8_t* mask, double* stat_sum,
                                unsigned long long* stat_count, hipStream_t s);
hipError_t launch_zero_words(void* p, int n, hipStream_t s);
hipError_t launch_active_list(int batch, int seq, int prefix, int32_t* act_idx, int32_t* act_off, hipStream_t s);
hipError_t launch_copy_rows(const void* src, void* dst, int n_rows, int row_bytes,
                            const int32_t* idx, const int32_t* m_dev, hipStream_t s);
// rows r = 0 .. n_rows-1; with seq > 0 row r is token (r / (seq - prefix)) * seq + prefix + r % (seq - prefix)
hipError_t launch_norm(int dtype, int kind, const void* x, const void* gain, const void* bias, float eps,
                       int n_rows, int d, void* out, int seq, int prefix, hipStream_t s);
hipError_t launch_residual_add(int dtype, const void* x, const void* o, void* out, long n_elems,
                               hipStream_t s);
// What launch_residual_norm does with the rows of a frozen prefix.  kLeftOut: rows as in launch_norm; else n_rows is all rows, and a
// frozen one gets the sum alone, or the norm of its x alone.  keep_x: the sums are stored.
enum class FrozenRows { kLeftOut, kSumOnly, kNormOnly };
hipError_t launch_residual_norm(int dtype, void* x, const void* o, const void* gain, float eps, int n_rows, int d,
                                void* h, int seq, int prefix, hipStream_t s, FrozenRows frozen_rows = FrozenRows::kLeftOut,
                                bool keep_x = true);
hipError_t launch_residual_rows(int dtype, void* x, const void* f, int n_rows, int d, const int32_t* idx,
                                hipStream_t s);
hipError_t launch_gather_rows(const void* src, void* dst, const int32_t* ids, int n_rows, int n_src,
                              int row_bytes, hipStream_t s);
hipError_t launch_swiglu(int dtype, void* gate, const void* up, int n_rows, int width, const int32_t* idx,
                         hipStream_t s);

// The attention block of dare_block_step without its first and last launch, for the model
// runtime, which fuses them with its neighbours: `h` is the hidden state already normalised,
// the block output O goes into o_cache only (no residual sum).  Arguments are checked as
// in dare_layer_step; rotary embedding as attached to the context.
// parts: the workspace of a step (its owner runs one step at a time), not the context's.
dare_status block_core(dare_ctx* ctx, int mode, float threshold, int batch, int seq, const void* h, float* q_prev,
                       void* k_cache, void* v_cache, void* o_cache, uint8_t* reuse_mask, int32_t* sel_count,
                       const AttnParts& parts, void* hip_stream);

// dare_create, optionally without the workspace of attention whose keys are cut: for contexts whose
// steps run through block_core.
dare_status create_context(const dare_config* cfg, const void* wq, const void* wk, const void* wv, const void* wo,
                           bool with_parts, void* hip_stream, dare_ctx** out_ctx);

}  // namespace dare
