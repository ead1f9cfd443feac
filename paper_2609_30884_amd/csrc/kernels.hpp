// Launchers of the device kernels (internal to libcrf.so).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "common.hpp"

namespace crf {

// ---------------------------------------------------------------- shared
// y = g * x / sqrt(mean(x^2) + eps) row-wise over d; x fp32 or bf16, y and g
// bf16.  copy_out (nullable) receives x as fp32.
hipError_t launch_rmsnorm(hipStream_t s, const void *x, bool x_f32, const void *g, bf16 *y, float *copy_out, int M,
                          int d, float eps);
// cos/sin table cs[p*hd/2 + i] = (cos, sin)(p * theta^(-2i/hd)), angles in fp64.
hipError_t launch_rope_table(hipStream_t s, float2 *cs, int T, int hd, float theta);

// ---------------------------------------------------------------- fp32 path
enum F32Epi { F32_QKV = 0, F32_RESID = 1, F32_SWIGLU = 2, F32_PLAIN = 3 };
// adapters up to this rank are formed inside the projection (one 16-row block)
constexpr int F32_FUSED_RANK = 16;
// Y = norm(x) W^T + adapter with one of the epilogues:
//   F32_QKV    rows [0, seg1) Q, [seg1, seg2) K, [seg2, N) V: bias, rotation, Q
//              to out, K and V to the pages of kv;
//   F32_RESID  out = resid_in + Y (either may be the other);
//   F32_SWIGLU out = silu(Y_0) * Y_1 of segments 0 (gate) and 1 (up);
//   F32_PLAIN  out = scale * Y (an adapter's U, for ranks past F32_FUSED_RANK).
struct F32Gemm {
  const float *x;
  int64_t ldx;
  int M, K, N;
  const float *gain;       // RMSNorm gain of x (nullable: x as it is), with eps
  float eps;
  const float *w[3];       // [seg_rows, K]
  int seg_rows[3];
  int seg1, seg2;
  int n_form;              // F32_QKV: rows with Q's, whether the launch has them or not
  // adapter of segment s: la [rank, K], lb [seg_rows, rank] (both null: none);
  // past F32_FUSED_RANK U [M, ldu] holds segment s's scaled U at column s * rank
  const float *la[3], *lb[3];
  int rank;
  float scale;
  const float *U;
  int ldu;
  float *out;
  int64_t ldo;
  const float *resid_in;
  const float *bias[3];
  const float2 *rope_cs;
  PagedKV kv;
  int hd;
};
hipError_t launch_gemm_f32(hipStream_t s, F32Epi epi, const F32Gemm &p);
hipError_t launch_attn_f32(hipStream_t s, const float *Q, const PagedKV &kv, float *O, int M, int nq, int nkv,
                           int hd);

// ---------------------------------------------------------------- bf16 path
struct LoraDownTarget {
  const bf16 *A;   // [rank, K] or nullptr
  int rank;
  float scale;
  int ucol;        // first column of this target in U
};
// U[m, ucol_t + j] = bf16(scale_t * sum_k X[m,k] A_t[j,k]) for j < rank_pad(t)
// (zero for rank <= j < rank_pad).
// With n_parts (M <= 16) U is not formed; unscaled fp32 parts of it are left in
// ws ([part][16][n_targets * rank_pad], ws_floats floats), *n_parts of them, for
// the projection to sum.  Without, `lw` (nullable blocks) lets K be split over
// workgroups, in `floats` floats and n_tickets counters that are zero between
// launches.
struct LoraWs {
  float *blocks = nullptr;
  int64_t floats = 0;
  unsigned *tickets = nullptr;
  int n_tickets = 0;
};
hipError_t launch_lora_down_bf16(hipStream_t s, const bf16 *X, int64_t ldx, int M, int K, const LoraDownTarget *t,
                                 int n_targets, int rank_pad, bf16 *U, int ldu, float *ws, int64_t ws_floats,
                                 int *n_parts, const LoraWs &lw);

enum GemmEpi { EPI_QKV = 0, EPI_RESID = 1, EPI_SWIGLU = 2 };

struct GemmParams {
  const bf16 *X;
  int64_t ldx;
  int M, K;
  int N;                       // rows of the (virtual) weight matrix in tile space
  const bf16 *w[3];            // segment row sources, each [rows, K]
  int seg1, seg2;              // EPI_QKV: first rows of the k and v segments
  // LoRA delta: acc += U[:, ucol_s : ucol_s + kpad] * lb_s^T  per segment s (few
  // token rows: U comes as upart below)
  const bf16 *U;
  int ldu, kpad, rank;
  const bf16 *lb[3];           // [seg_rows, rank] or nullptr
  int ucol[3];
  // EPI_QKV
  const bf16 *bias[3];
  bf16 *q_out;
  int dq, hd;
  float q_scale;               // factor applied to Q (after bias and rotary) before it is stored
  PagedKV kv;
  const float2 *rope_cs;
  // EPI_QKV: token row m sits at position pos0 + m (rotary angle and page slot)
  int pos0;
  // EPI_RESID: resid[m, n] += acc (= acc when resid_overwrite); resid_out (nullable) = bf16(resid)
  float *resid;
  // EPI_RESID (nullable): the residual before the update in bf16, same layout
  // as resid, read instead of resid (the window's first update reads its
  // boundary state directly, so the fp32 copy of it is never written)
  const bf16 *resid_in;
  bf16 *resid_out;
  int resid_final;  // EPI_RESID with resid_out: the updated residual is stored only as resid_out
  int ldr;
  int resid_overwrite;
  // EPI_SWIGLU: act[m, f] = silu(gate) * up
  bf16 *act;
  int d_ffn;
  // few token rows: U given as unscaled K-split parts ([part][16][upart_cols]
  // fp32, upart_n > 0 parts) to be summed, scaled by uscale and rounded to bf16
  const float *upart;
  int upart_n, upart_cols;
  float uscale;
  // EPI_RESID, EPI_QKV: when the tiles leave the last wave of the grid at most
  // half full (n_cu compute units; two thirds with a long K), the last tiles are
  // split into K-parts that write fp32 partials to split_part (split_cap floats)
  // and a second kernel adds them up in a fixed order.  split_first / split_s are
  // set by the launcher.
  float *split_part;
  int64_t split_cap;
  // few token rows: arrival counters of K-split workgroups, zero between launches
  unsigned *tickets;
  int n_tickets;
  int kpairs;  // pairs of k-steps per part, set by the launcher
  int n_cu;
  int split_first, split_s;
  // EPI_SWIGLU: the down projection's adapter down-projection fused into the
  // epilogue (rank <= 16): dn_a = A_down [dn_rank, d_ffn].  Each workgroup sums
  // act . A_down^T over the features of consecutive items on one token tile (a
  // run) and leaves the sums in dn_part slot b * dn_runs + run ([slot][2][256][16]
  // fp32); dn_head[tm * tiles_n + tn] = slot + 1 for the first tile of a run,
  // else 0.  launch_gemm_dn_sum then forms U.
  const bf16 *dn_a;
  int dn_rank;
  float *dn_part;
  int *dn_head;
  int dn_runs;
};
// Persistent over at most n_cu workgroups (n_cu > 0).  *dn_done (nullable)
// reports whether the fused down-projection sums were produced (they are
// skipped when a workgroup would need more than dn_runs runs).
hipError_t launch_gemm_bf16(hipStream_t s, GemmEpi epi, int hd, const GemmParams &p, bool *dn_done = nullptr);
// U[m, ucol + r] = bf16(scale * sum of the fused sums) for r < dn_rank, after
// launch_gemm_bf16(EPI_SWIGLU) reported *dn_done with the same parameters.
hipError_t launch_gemm_dn_sum(hipStream_t s, const GemmParams &p, bf16 *U, int ldu, int ucol, float scale);
// The same projections for M <= 16 token rows (weight-streaming bound).
hipError_t launch_gemm_skinny_bf16(hipStream_t s, GemmEpi epi, const GemmParams &p);
// y = RMSNorm(x) g of up to 16 rows (copy_out, nullable, receives x in fp32)
// with the adapters' down-projection of y: part[s][16][n_blocks * 16] unscaled,
// s < norm_lora_parts(d); n_blocks = targets * rank_pad / 16 (0: no adapter).
struct NormLora {
  const void *x;
  const bf16 *g;
  bf16 *y;
  float *copy_out;
  int M, d;
  float eps;
  const bf16 *A[3];  // [rank, d] or null
  int rank, rank_pad;
  float *part;
};
int norm_lora_parts(int d);
hipError_t launch_norm_lora(hipStream_t s, bool x_f32, const NormLora &p, int n_blocks);

// ---- 17 token rows and more (13 with large adapters), up to where the 256x256 tiles win (gemm_mid.hip)
constexpr int MID_SEGS = 6;       // row sources of a launch: up to three weights, then their A factors
constexpr int MID_MAX_COLS = 8192;  // widest residual row of reduce_resid
// Y = X W^T over the concatenated rows [0, N) of the segments (each a multiple
// of 8 rows): fp32 K-parts part[s][m][n], s < parts; or for gate/up (segments 0
// and 1 in tile space, N = 2 d_ffn, parts = 1) act = silu(gate) * up.
struct MidGemm {
  const bf16 *X;
  int64_t ldx;
  int M, K, N;
  const bf16 *w[MID_SEGS];
  int w_rows[MID_SEGS], seg_end[MID_SEGS];  // rows of a segment; first row after it
  int parts, tiles_m;  // tiles_m is set by the launcher
  float *part;
  // gate/up: adapter delta U lb^T and the output
  const bf16 *U;
  int ldu, rank, ucol[2];
  const bf16 *lb[2];
  bf16 *act;
  int d_ffn;
};
// K-parts that fill the GPU for a product of N rows, within part_floats floats
int mid_parts(int M, int N, int K, int n_cu, int64_t part_floats);
hipError_t launch_gemm_mid(hipStream_t s, bool gate_up, const MidGemm &p);
// Sums the parts of [M, ld] (n_base base columns, then n_u adapter columns) and
// finishes the projection of each token (see gemm_mid.hip).
struct MidReduce {
  const float *part;
  int parts, M, ld, n_base, n_u;
  float scale;             // of the adapter
  int rank, ucol[3];       // columns of the targets' U among the n_u
  const bf16 *lb[3];       // [rows, rank] or null
  // QKV: segments [0, seg1) Q, [seg1, seg2) K, [seg2, n_base) V
  int seg1, seg2, hd, dq, pos0;
  float q_scale;
  const bf16 *bias[3];
  bf16 *q_out;
  PagedKV kv;
  const float2 *rope_cs;
  // residual rows: resid (fp32) += sum, the old value from resid_in when given;
  // resid_out (nullable) takes the result in bf16 instead; with a gain, xn =
  // RMSNorm of the result
  float *resid;
  const bf16 *resid_in;
  bf16 *resid_out;
  const bf16 *gain;
  float eps;
  bf16 *xn;
};
hipError_t launch_mid_reduce_qkv(hipStream_t s, const MidReduce &p);
hipError_t launch_mid_reduce_resid(hipStream_t s, const MidReduce &p);

// Factor the attention kernel expects the stored query rows to carry:
// log2(e) / sqrt(head_dim) (scores then come out in log2 units).
inline float attn_query_scale(int hd) { return 1.4426950408889634f / __builtin_sqrtf((float)hd); }
// Query rows 0..Mq-1 at positions q_off..q_off+Mq-1 over keys 0..q_off+Mq-1,
// Q pre-multiplied by attn_query_scale(hd).
// part (nullable, part_floats floats): workspace for splitting the keys over
// workgroups: of a few query rows or blocks over a long prefix, or of a window's
// longest blocks.  With `lora` (Mq <= 16) and a
// split launch the merge also forms the parts of O A^T, one per query head
// (lora->n_parts set; else it stays 0).
struct AttnLora {
  const bf16 *A;   // [rank, nq * hd]
  int rank, cols;  // part[head][16][cols]
  float *part;
  int n_parts;
};
hipError_t launch_attn_bf16(hipStream_t s, const bf16 *Q, const PagedKV &kv, bf16 *O, int Mq, int q_off, int nq,
                            int nkv, int hd, float *part, int64_t part_floats, AttnLora *lora = nullptr);

// ---------------------------------------------------------------- drift
// One factor tensor of the current adapter; the same tensor of the stored
// version v is b[seg * n_versions + v] of the launch.
struct DriftSeg {
  const void *a;
  int64_t count;     // elements
};
struct DriftChunk {
  int seg, idx;      // elements [idx * chunk, (idx + 1) * chunk) of the segment
};
struct DriftArgs {
  const DriftSeg *segs;
  const void *const *b;
  const DriftChunk *chunks;      // layer by layer
  int n_chunks, chunk;           // chunk: elements, a multiple of 4096
  const int *first;              // [n_layers + 1] first chunk of a layer
  const int *anchor;             // [n_layers]
  int n_versions, n_layers;
  unsigned *ticket;              // zero at launch
  double *partials;              // [n_versions][n_chunks]
  double *sq;                    // [n_versions][n_layers] (workspace)
  const float *sens;
  int per_layer_only;
  float *drift, *risk, *sq_out;  // sq_out nullable
};
// Device address of the no-allocation drift scratch on the current device
// (CRF_DRIFT_NOALLOC_MAX_BYTES, looked up once per device).
hipError_t drift_noalloc_scratch(void **out);
hipError_t launch_drift(hipStream_t s, bool f32, const DriftArgs &a);

}  // namespace crf
