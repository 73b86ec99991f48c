// Internal launch interface between the C-ABI layer and the kernel files.
// Every launcher enqueues on `st` and returns; shapes were validated by the caller.
#pragma once

#include "poetx_common.h"

namespace poetx {

// Brackets the launches of one stage with HIP events when stage profiling is on.
class StageTimer {
 public:
  StageTimer(int stage, hipStream_t st);
  ~StageTimer();
 private:
  hipStream_t st_;
  long idx_;
};

// ---- plain fp32-FMA path (fma_kernels.hip): any dtype, any block size ---------------
// out = op(W) * act:  W is n x m row major.  trans_w == 0: out (n x N) = W act (m x N);
// trans_w == 1: out (m x N) = W^T act (n x N).
void fma_dense(int dtype, int trans_w, const void* W, int n, int m, const void* act, void* out,
               i64 N, hipStream_t st);
// V: d x cols, out: d x cols_out (the columns past cols are written as zeros)
void fma_apply_left(int dtype, const void* V, i64 ldv, i64 cols, void* out, i64 ldo, i64 cols_out, int d, const int32_t* perm, const void* blocks,
                    int b, int transpose_G, hipStream_t st);
// is that faster than the edge kernel?
bool fma_apply_left_preferred(int d, i64 cols, int b);
void fma_apply_right(int dtype, const void* V, void* out, i64 rows, int d, i64 ld, const int32_t* perm,
                     const void* blocks, int b, int transpose_G, hipStream_t st);
// dG[j] = U'_j V'_j^T with rows of U and V (d x N each) gathered by perm; dG is [nb][b][b] float.
void fma_blockgrad(int dtype, const void* U, const void* V, int d, i64 N, const int32_t* perm, int b,
                   float* dG, hipStream_t st);
// ws: 2 * nb*b*b floats.
void fma_cnp_build(const float* theta, int d, int b, int k, float* G_f32, void* E_bf16, float* ws,
                   hipStream_t st);
// dG -> dtheta.  ws: 4 * nb*b*b floats.
void fma_cnp_bwd(const float* theta, const float* dG, int d, int b, int k, float* dtheta, int accumulate,
                 float* ws, hipStream_t st);

// ---- edge-handling matrix-core path (edge.hip): bf16 and fp32, any sizes, strides and alignments --------
// ws: the bytes the queries report (fp32 partials of a split contraction; 0 where there is no split).
// act has act_cols columns, which the plan is made for and the query is asked with; the first N of the product go to out.
// aligned: may both operands lie on 16-byte boundaries (not where such a product runs on another kernel)?
size_t edge_dense_workspace_bytes(int dtype, int trans_w, int n, int m, i64 act_cols, bool aligned);
void edge_dense(int dtype, int trans_w, const void* W, int n, int m, const void* act, i64 ld_act, i64 act_cols, void* out, i64 ld_out, i64 N,
                void* ws, hipStream_t st);
// V: d x cols, out: d x cols_out (cols_out >= cols; the extra columns are written as zeros); plan_cols: columns to choose the tile for
void edge_apply_left(int dtype, const void* V, i64 ldv, void* out, i64 ldo, int d, i64 cols, i64 cols_out, i64 plan_cols, const int32_t* perm,
                     const void* blocks, int b, int transpose_G, hipStream_t st);
// does edge_apply_left take its smallest tile?
bool edge_apply_smallest_tile(int d, i64 plan_cols, int b);
// the same on that tile for a few tokens with exactly one of V, out token major ([token][ld])
void edge_apply_tokens(int dtype, const void* V, i64 ldv, bool v_tm, void* out, i64 ldo, bool out_tm, int d, i64 cols, i64 cols_out,
                       const int32_t* perm, const void* blocks, int b, int transpose_G, hipStream_t st);
// Block gradients over N tokens.  cols_u, cols_v: columns that the operands have, those past N being zeros (of a feature whose weights are
// not finite also NaN: its tokens are not finite either).  parts: the sums of token ranges, each ceil(d/b) * b * b floats, one after the other.
struct GradProblem {
  const void* U;
  const void* V;
  i64 ldu, cols_u, ldv, cols_v, N;
  int d;
  const int32_t* perm;
  float* parts;
};
size_t edge_blockgrad_workspace_bytes(int dtype, int d, i64 N, int b);
void edge_blockgrad(int dtype, GradProblem q, int b, float* dG, void* ws, hipStream_t st);   // summed up (parts is not used)
// both sides of a layer (b * b a multiple of four)
size_t edge_blockgrad_pair_workspace_bytes(int dtype, int d0, int d1, i64 N, int b);
void edge_blockgrad_pair(int dtype, GradProblem q0, GradProblem q1, int b, float* dG0, float* dG1, void* ws, hipStream_t st);
// The same, left as its parts; returns how many.
size_t edge_blockgrad_parts_bytes(int dtype, int d, i64 N, int b);
int edge_blockgrad_parts(int dtype, const GradProblem& q, int b, hipStream_t st);
// both sides of a layer, in one launch where their plans allow
void edge_blockgrad_parts_pair(int dtype, const GradProblem& q0, const GradProblem& q1, int b, int* n0, int* n1, hipStream_t st);
// ... and, in the same launch, out = op(blocks) V on q1's side: where the first says so
bool edge_apply_joins_blockgrads(int dtype, int d_apply, i64 plan_cols, int d0, int d1, i64 N, int b);
void edge_apply_blockgrad_parts(int dtype, const void* V, i64 ldv, void* out, i64 ldo, i64 cols, i64 cols_out, i64 plan_cols, const void* blocks, const GradProblem& q0,
                                const GradProblem& q1, int b, int* n0, int* n1, hipStream_t st);

// ---- the forward of up to 32 bf16 tokens (few_tokens.hip); tensors of any alignment ----------
bool few_tokens_supported(int n, int m, int b, i64 N);
// V, out: feature major (row stride ld) or token major ([token][ld]); not V token major with out feature major
void few_apply(const void* V, i64 ldv, bool v_tm, void* out, i64 ldo, bool out_tm, int d, int N, const int32_t* perm, const void* E, int b, int trans,
               hipStream_t st);
// out (M x cols feature major, columns from N on zero) = W (M x K) times act ([token][K])
void few_dense(const void* W, int M, int K, const void* act, void* out, i64 ldo, int N, int cols, hipStream_t st);

// ---- fp32 series of blocks up to 128, one launch (series_small.hip) ----------------------------------------
bool series_small_supported(int b);
void series_small_build(const float* theta, int d, int b, int k, float* G_f32, void* E_bf16, hipStream_t st);
struct SeriesSide {
  const float* theta;
  const float* dG;        // nsplit block gradients of ceil(d/b) * b * b floats, split_stride floats apart, that add up to dL/dG
  i64 split_stride;
  int nsplit, d;
  float* dtheta;
};
void series_small_bwd(const SeriesSide* sides, int nsides, int b, int k, int accumulate, hipStream_t st);   // one or two sides

// dtheta[j][idx(i,c)] (+)= M[j][i][c] - M[j][c][i] (Sec. 3.4: gradient on the packed parameters).
void skew_project_launch(const float* M, int b, int d, float* dtheta, int accumulate, hipStream_t st);

// ---- INT8 base weight (weight_q8.hip): codes [n][m] then, 256-byte aligned, float scale[n]
size_t weight_q8_scale_offset(int n, int m);
void weight_quantize_q8_launch(int dtype, const void* W, int n, int m, void* Wq, hipStream_t st);
void weight_dequantize_q8_launch(const void* Wq, int n, int m, int dtype, void* W_out, hipStream_t st);

// out (C x R_out, row stride ld_out) = in (R x C, row stride ld_in)^T, columns R .. R_out - 1 of out zero (layout.hip)
void transpose_launch(int dtype, const void* in, void* out, i64 R, i64 C, i64 ld_in, i64 ld_out, i64 R_out, hipStream_t st);

void perm_validate_launch(const int32_t* perm, int d, int32_t* scratch, hipStream_t st);

// ---- matrix-core path for bf16 (mfma_*.hip) -------------------------------------------
bool mfma_dense_supported(int n, int m, i64 N);
// act: K x N_act dense (whole tiles); the first N columns of the product go to out (row stride ld_out, any alignment
// where N < N_act).  ws: the bytes the query reports (M, N_act, K of the product; parts of a split contraction).
size_t mfma_dense_workspace_bytes(i64 M, i64 N, i64 K);
void mfma_dense(int trans_w, const void* W, int n, int m, const void* act, i64 N_act, void* out, i64 ld_out, i64 N, void* ws, hipStream_t st);
int mfma_dense_splits(i64 M, i64 N, i64 K);   // contraction ranges of that product
void mfma_dense_reduce(const float* parts, int splits, i64 M, i64 Np, void* out, i64 ld_out, i64 N, hipStream_t st);
// is a ragged token count better padded to whole tiles for the streaming product than left to the edge one?
bool mfma_dense_worth_padding(int n, int m, i64 N);
// the same products for fp32 tensors (fp32 MFMA, mfma_dense_f32.hip)
bool mfma_dense_f32_supported(int n, int m, i64 N);
bool mfma_dense_f32_preferred(int n, int m, int M, i64 N);
void mfma_dense_f32(int trans_w, const void* W, int n, int m, const void* act, void* out, i64 N, hipStream_t st);
// the same products on a quantised weight buffer (codes + row scales), dequantised inside the kernel (mfma_dense_q8.hip)
bool mfma_dense_q8_supported(int n, int m, i64 N);
void mfma_dense_q8(int trans_w, const void* Wq, int n, int m, const void* act, void* out, i64 N, void* ws, hipStream_t st);   // ws as mfma_dense
bool mfma_apply_left_supported(int d, i64 cols, i64 ld, int b);
void mfma_apply_left(const void* V, void* out, int d, i64 cols, i64 ld, const int32_t* perm,
                     const void* E, int b, int transpose_G, hipStream_t st);
// the same for any token counts and row strides (element-aligned activations, 16-byte aligned blocks): V d x cols, out d x cols_out,
// columns past cols written as zeros
bool mfma_apply_left_ragged_supported(int d, i64 cols_out, int b);
void mfma_apply_left_ragged(const void* V, i64 ldv, i64 cols, void* out, i64 ldo, i64 cols_out, int d, const int32_t* perm, const void* E, int b,
                            int transpose_G, hipStream_t st);
bool mfma_blockgrad_supported(int d, i64 N, int b);
bool mfma_blockgrad_preferred(int d, i64 N, int b);   // ... and large enough for it
size_t mfma_blockgrad_workspace_bytes(int d, i64 N, int b);
// U and V: d rows of at least N tokens, row strides multiples of 8
void mfma_blockgrad(const void* U, i64 ldu, const void* V, i64 ldv, int d, i64 N, const int32_t* perm, int b, float* dG, void* ws, hipStream_t st);
// One pass over the incoming gradient V (d x N) for one side (mfma_applygrad.hip, b = 256):
// out = Psi^T Diag(op(G)) Psi V and dG[j] = U'_j V'_j^T (rows gathered by perm).  ws: the bytes the
// query reports (partial block gradients of the token ranges).
bool mfma_apply_grad_supported(int d, i64 N, i64 ld, int b);
size_t mfma_apply_grad_workspace_bytes(int d, i64 N);
void mfma_apply_grad(const void* V, const void* U, void* out, int d, i64 N, i64 ld, const int32_t* perm, const void* E,
                     int transpose_G, float* dG, void* ws, hipStream_t st);
bool mfma_cnp_supported(int d, int b);
void mfma_cnp_build(const float* theta, int d, int b, int k, float* G_f32, void* E_bf16, float* ws,
                    hipStream_t st);
// One or two sides whose dG (one matrix per block, nsplit = 1) follow each other in memory; ws: 5 floats per element
// (tiled), 2 (on chip).
void mfma_cnp_bwd(const SeriesSide* sides, int nsides, int b, int k, int accumulate, float* ws, hipStream_t st);
// b = 256: whole chain of a block in one launch, block resident on chip (mfma_cnp_lds.hip).
bool lds_cnp_supported(int d, int b);
void lds_cnp_build(const float* theta, int nb, int k, float* G_f32, void* E_bf16, float* ws, hipStream_t st);   // ws: half a float per block element
// Backward of one or two sides (dG of a side: one matrix per block, nsplit = 1).  ws: 2 floats per block element.
void lds_cnp_bwd(const SeriesSide* sides, int nsides, int k, int accumulate, float* ws, hipStream_t st);
// b = 256, nb0 + nb1 blocks of two sides: bf16(Q), or where dL/dG is given bf16(-Q) and bf16(dL/dG), as the chains' fragments; and their dL/dQ (tiles
// in the chains' order) -> packed gradients (skew_tiled.hip)
void skew_materialize_chain_launch(const float* theta0, i64 nb0, const float* theta1, i64 nb1, uint16_t* Qf, const float* D0, const float* D1, uint16_t* Df,
                                   hipStream_t st);
void skew_project_chain_launch(const float* M, i64 nb0, float* dtheta0, i64 nb1, float* dtheta1, int accumulate, hipStream_t st);
// dL/dQ of nb0 + nb1 blocks -> packed gradients of two sides (skew_tiled.hip)
void skew_project_sides_launch(const float* M, int b, i64 nb0, float* dtheta0, i64 nb1, float* dtheta1, int accumulate, hipStream_t st);
// Through 64 x 64 tiles, coalesced on both sides of the transpose (skew_tiled.hip): Q of nb blocks from packed parameters, Qf fp32, Qb bf16,
// Tb = bf16(-Q), [nb][b][b] (any may be null); and the projection.
bool skew_tiled_supported(int b, i64 d);
void skew_materialize_tiled_launch(const float* theta, int b, i64 nb, float* Qf, uint16_t* Qb, uint16_t* Tb, hipStream_t st);
void skew_project_tiled_launch(const float* M, int b, i64 nb, float* dtheta, int accumulate, hipStream_t st);

}  // namespace poetx
