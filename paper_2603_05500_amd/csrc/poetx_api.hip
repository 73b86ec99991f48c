// C-ABI entry points: host-side argument checks and kernel dispatch.
// Every step of the path runs in the kernels of this library; this file only
// validates, carves the workspace and enqueues.
#include <atomic>
#include <mutex>

#include "poetx_kernels.h"

using namespace poetx;

namespace {

std::atomic<int> g_force_fma{0};

// ---- scratch of the entry point that allocates nothing (poetx_cnp_build_static) ------------
// One copy of this array lives on every GPU the library runs on, for as long as the process
// lives.  Its name is only a host-side handle: kernels get the per-device address that
// hipGetSymbolAddress returns, looked up once per device with that device current.
constexpr size_t kStaticCnpElems = POETX_CNP_STATIC_MAX_ELEMS;           // block elements: ceil(d/b) * b * b
constexpr size_t kStaticCnpBytes = 12 * kStaticCnpElems;                 // poetx_cnp_workspace_bytes per element
static __device__ __align__(256) unsigned char scratch[kStaticCnpBytes];
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

int static_scratch(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return POETX_ERR_HIP;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return POETX_ERR_HIP;
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return POETX_OK;
}

inline bool use_mfma(int dtype) { return dtype == POETX_BF16 && !g_force_fma.load(); }
// series of small blocks: fp32 whatever the precision asked for, one launch for a whole chain
inline bool series_small(int b) { return series_small_supported(b) && !g_force_fma.load(); }
// the streaming kernels move 16 bytes per lane: every tensor they touch must be 16-byte aligned
inline bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }
inline size_t esize(int dtype) { return dtype == POETX_F32 ? 4 : 2; }
inline bool dtype_ok(int dtype) { return dtype == POETX_F32 || dtype == POETX_BF16; }
inline bool overlap(const void* a, size_t na, const void* b, size_t nb) {
  const char* x = (const char*)a;
  const char* y = (const char*)b;
  return x < y + nb && y < x + na;
}

int check_desc(const poetx_linear_desc* d) {
  if (!d) return POETX_ERR_INVALID_ARG;
  if (d->d_in <= 0 || d->d_out <= 0 || d->block <= 0 || d->neumann_k < 1 || d->n_tokens <= 0)
    return POETX_ERR_INVALID_ARG;
  if (!dtype_ok(d->dtype)) return POETX_ERR_INVALID_ARG;
  if (d->cnp_precision != POETX_CNP_FP32 && d->cnp_precision != POETX_CNP_BF16) return POETX_ERR_INVALID_ARG;
  if ((d->flags & ~(POETX_FLAG_RECOMPUTE_B | POETX_FLAG_W_INT8 | POETX_FLAG_BLOCK_GRADS | POETX_FLAG_W_INT8_FUSED)) != 0 || (d->layout != POETX_FEATURE_MAJOR && d->layout != POETX_TOKEN_MAJOR))
    return POETX_ERR_INVALID_ARG;
  if ((d->flags & POETX_FLAG_W_INT8) && !(d->flags & POETX_FLAG_RECOMPUTE_B)) return POETX_ERR_INVALID_ARG;
  if ((d->flags & POETX_FLAG_W_INT8_FUSED) && !(d->flags & POETX_FLAG_W_INT8)) return POETX_ERR_INVALID_ARG;
  if (d->block > d->d_in || d->block > d->d_out) return POETX_ERR_BAD_SHAPE;
  if (d->n_tokens >= (1ll << 31) || (i64)d->n_tokens * (d->d_in > d->d_out ? d->d_in : d->d_out) >= (1ll << 40))
    return POETX_ERR_UNSUPPORTED;
  return POETX_OK;
}

// dG plus the chain's scratch of nb blocks.  The b = 512 chain lays out five floats per element, the plain one four, the on-chip one of b = 256 two;
// what k + 2 > 5 reserves beyond that is slack, left as it has always been reported.
size_t cnp_bwd_ws_floats(i64 nb, int b, int k) {
  const size_t elems = (size_t)nb * b * b;
  return elems + (size_t)(k + 2 > 5 ? k + 2 : 5) * elems;
}
// ... of a call's series: those of one side after the other, or of both sides together
size_t cnp_bwd_ws_floats(const poetx_linear_desc* d) {
  return cnp_bwd_ws_floats((i64)ceil_div(d->d_in, d->block) + ceil_div(d->d_out, d->block), d->block, d->neumann_k);
}

// A d x cols activation, row stride ld.  Activations in the workspace have internal_columns() columns, the ones past
// the call's tokens being zeros (zeros stay zeros through every stage), so that the streaming kernels can run on whole
// tiles whatever the token count; a caller's tensors have exactly its tokens.
struct Act {
  const void* p;
  i64 ld, cols;
  void* out() const { return const_cast<void*>(p); }
};
inline i64 min64(i64 a, i64 b) { return a < b ? a : b; }

// Which kernels run an apply is decided before the tensors of a call are looked at (apply_streams below): in one pass some
// of them have padded columns and some do not, in another layout others, and the results are the same bit for bit.
// streams: the streaming kernels, whole tiles or not.  plan_cols: columns that the choice between the others, and their tile, is made for.
void apply_left_dispatch(int dtype, const Act& V, const Act& out, int d, const int32_t* perm, const void* blocks, int b, int trans, bool streams,
                         i64 plan_cols, hipStream_t st) {
  StageTimer tm(POETX_STAGE_APPLY, st);
  if (use_mfma(dtype) && streams && aligned16(blocks)) {
    if (V.ld == out.ld && V.cols == out.cols && mfma_apply_left_supported(d, V.cols, V.ld, b) && aligned16(V.p) && aligned16(out.p))
      mfma_apply_left(V.p, out.out(), d, V.cols, V.ld, perm, blocks, b, trans, st);
    else
      mfma_apply_left_ragged(V.p, V.ld, min64(V.cols, out.cols), out.out(), out.ld, out.cols, d, perm, blocks, b, trans, st);
  } else if (!g_force_fma.load() && !fma_apply_left_preferred(d, plan_cols, b)) {
    edge_apply_left(dtype, V.p, V.ld, out.out(), out.ld, d, min64(V.cols, out.cols), out.cols, plan_cols, perm, blocks, b, trans, st);
  } else {
    fma_apply_left(dtype, V.p, V.ld, min64(V.cols, out.cols), out.out(), out.ld, out.cols, d, perm, blocks, b, trans, st);
  }
}
// an apply on its own: V and out of one shape
void apply_left_alone(int dtype, const Act& V, const Act& out, int d, const int32_t* perm, const void* blocks, int b, int trans, hipStream_t st) {
  const bool whole = mfma_apply_left_supported(d, V.cols, V.ld, b) && aligned16(V.p) && aligned16(out.p);
  apply_left_dispatch(dtype, V, out, d, perm, blocks, b, trans, whole || mfma_apply_left_ragged_supported(d, V.cols, b), V.cols, st);
}

// part: scratch of dense_part_bytes() for products that split their contraction.
// w_q8: W is a quantised weight buffer that the product dequantises itself (see weight_in_kernel)
// As with the applies the kernel follows from the descriptor: the plan from the activation operand, which is always a workspace
// one, the fp32 kernel from the call's own tokens (whole tiles of those leave no tensor padded).
void dense_dispatch(const poetx_linear_desc* desc, int trans_w, const void* W, const Act& act, const Act& out, void* part, hipStream_t st,
                    bool w_q8) {
  StageTimer tm(POETX_STAGE_DENSE, st);
  const int dtype = desc->dtype, n = desc->d_out, m = desc->d_in;
  const i64 N = min64(act.cols, out.cols);
  if (w_q8) mfma_dense_q8(trans_w, W, n, m, act.p, out.out(), N, part, st);
  else if (use_mfma(dtype) && act.ld == act.cols && mfma_dense_supported(n, m, act.cols) && aligned16(W) && aligned16(act.p))
    mfma_dense(trans_w, W, n, m, act.p, act.cols, out.out(), out.ld, N, part, st);
  else if (dtype == POETX_F32 && !g_force_fma.load() && mfma_dense_f32_preferred(n, m, trans_w ? m : n, desc->n_tokens) && aligned16(W) && aligned16(act.p) &&
           aligned16(out.p))
    mfma_dense_f32(trans_w, W, n, m, act.p, out.out(), N, st);
  else if (!g_force_fma.load()) edge_dense(dtype, trans_w, W, n, m, act.p, act.ld, act.cols, out.out(), out.ld, N, part, st);
  else fma_dense(dtype, trans_w, W, n, m, act.p, out.out(), N, st);
}

// POET-XQ: do the dense kernels read the 8-bit weight directly (conversion inside the operand path; asked for
// with POETX_FLAG_W_INT8_FUSED)?  Otherwise the weight is dequantised into the workspace before the products.
bool weight_in_kernel(const poetx_linear_desc* d) {
  return (d->flags & POETX_FLAG_W_INT8) && (d->flags & POETX_FLAG_W_INT8_FUSED) && use_mfma(d->dtype) && mfma_dense_q8_supported(d->d_out, d->d_in, d->n_tokens);
}

// Columns of the activations in the workspace.  Shapes whose dense products the streaming kernel takes but for the token
// count are padded to its 256-token tiles (see dense_worth_padding for when that pays); others to whole 16-byte
// vectors, so that rows stay aligned.
i64 internal_columns(const poetx_linear_desc* d) {
  const i64 N = d->n_tokens;
  if (g_force_fma.load()) return N;                     // the plain kernels know one token count only
  const i64 Np = (N + 255) / 256 * 256;
  if (N == Np || N > (1ll << 31) - 256) return N;       // column counts are ints
  if (d->dtype == POETX_BF16 && mfma_dense_supported(d->d_out, d->d_in, Np) && mfma_dense_worth_padding(d->d_out, d->d_in, N)) return Np;
  return (N + 7) / 8 * 8;
}

// Do the applies of a layer's side take the streaming kernels (bf16)?  Whole tiles of the call's own tokens, or enough columns in
// the workspace.  The same answer for every tensor of every call on this descriptor, whatever its layout.
bool apply_streams(const poetx_linear_desc* d, int dim) {
  return mfma_apply_left_supported(dim, d->n_tokens, d->n_tokens, d->block) || mfma_apply_left_ragged_supported(dim, internal_columns(d), d->block);
}
void apply_left(const poetx_linear_desc* desc, const Act& V, const Act& out, int d, const int32_t* perm, const void* blocks, int trans, hipStream_t st) {
  apply_left_dispatch(desc->dtype, V, out, d, perm, blocks, desc->block, trans, apply_streams(desc, d), desc->n_tokens, st);
}

// Does poetx_linear_bwd stream each side's gradient once (aligned tensors)?  Not a short stream: the two halves' smaller tiles and both gradients in a launch are sooner done, the more so
// the more alike the sides are, as their gradients then share the launch evenly.  us without the series, one pass / two halves, by (d_in + d_out) N in units of 2^21: equal sides 3: 2048 x 2048 64 / 55;
// 4: 1024 x 1024 60 / 56, 2048 x 2048 64 / 59, 4096 x 4096 79 / 76; 5: 70 / 72, 75 / 79, 95 / 99; 15/16 to 3/4: 2048 x 1792 3.3: 66 / 55, 3.8: 62 / 57, 4.7: 74 / 78; 4096 x 3840 3.9: 78 / 75, 4.8: 92 / 98;
// 4096 x 3072 3.5: 73 / 70, 4.4: 80 / 83; a half and less: 2048 x 1024 2.6: 64 / 57, 3: 59 / 59, 3.8: 62 / 65; 4096 x 2048 3: 69 / 68, 3.8: 73 / 76; 4096 x 1024 2.5: 61 / 58, 3.1: 65 / 67.  Sides of ratios between
// 1/2 and 3/4 were not measured.
bool bwd_one_pass(const poetx_linear_desc* d) {
  const i64 N = d->n_tokens, wide = d->d_in > d->d_out ? d->d_in : d->d_out, narrow = d->d_in + (i64)d->d_out - wide;
  const bool alike = 3 * narrow > 2 * wide;
  return (wide + narrow) * N > (alike ? 4 : 3) << 21 && d->cnp_precision == POETX_CNP_BF16 && use_mfma(d->dtype) && lds_cnp_supported(d->d_in, d->block) && lds_cnp_supported(d->d_out, d->block) &&
         internal_columns(d) == N && mfma_apply_grad_supported(d->d_in, N, N, d->block) && mfma_apply_grad_supported(d->d_out, N, N, d->block);
}

// Few token-major tokens outside few_tokens(): the forward's applies read X and write Z as they are, element by element, where the two
// transposing launches (some 5 us each) would cost more.  Every 32 rows of a block read the whole block's features
// again, so the element reads are in proportion to (n + m) N b; the workgroups of b = 512 are besides a chain of four
// dependent stages, and lose from half of that on.  Forwards, us, with transposes / in place: bf16 512 x 1376, b = 64: 24.5 / 16.4 for one token, 26.1 / 20.8 for 16,
// 28.5 / 24.2 for 200; 480 x 960, b = 96: 24.0 / 16.1, 26.3 / 21.9, 27.0 / 23.7; 1024 x 1024, b = 128, 33 tokens 27.3 / 23.0, 100: 28.4 / 24.0 (128 tokens, before: 21.8 / 25.2,
// as bf16 transposes of whole 64-token tiles are half as dear); fp32 512 x 768, b = 64: 26.3 / 16.0, 25.9 / 16.0, 29.8 / 21.1; 2048 x 2048, b = 256: 37.9 / 27.5, 38.7 / 29.8;
// 4096 x 4096, b = 512: 61.9 / 54.4, three tokens 62.9 / 59.0, 16: 62.8 / 64.0.
bool reads_tokens_in_place(const poetx_linear_desc* d) {
  if (d->layout != POETX_TOKEN_MAJOR || g_force_fma.load()) return false;
  const i64 N = d->n_tokens;
  if (d->dtype == POETX_BF16 && N % 64 == 0) return false;
  if (use_mfma(d->dtype) && (apply_streams(d, d->d_in) || apply_streams(d, d->d_out))) return false;
  // the same kernel and tile as feature-major calls take: results are the same bit for bit in either layout
  if (fma_apply_left_preferred(d->d_in, N, d->block) || fma_apply_left_preferred(d->d_out, N, d->block)) return false;
  if (!edge_apply_smallest_tile(d->d_in, N, d->block) || !edge_apply_smallest_tile(d->d_out, N, d->block)) return false;
  return (double)(d->d_in + (i64)d->d_out) * N * d->block <= (d->block <= 256 ? 1 << 25 : 1 << 24);
}

// A handful of tokens: the forward's own short kernels, in every call that computes A and B (few_tokens_supported says where it pays).
bool few_tokens(const poetx_linear_desc* d) { return use_mfma(d->dtype) && few_tokens_supported(d->d_out, d->d_in, d->block, d->n_tokens); }
// B = W R^T X on them; A: scratch of n_tokens * d_in elements
void few_b(const poetx_linear_desc* d, const void* X, const void* W, const int32_t* perm_R, const void* blocks_R, const Act& A, const Act& B, hipStream_t st) {
  const bool tm = d->layout == POETX_TOKEN_MAJOR;
  const int N = (int)d->n_tokens;
  {
    StageTimer tim(POETX_STAGE_APPLY, st);
    few_apply(X, tm ? d->d_in : N, tm, A.out(), d->d_in, true, d->d_in, N, perm_R, blocks_R, d->block, 1, st);
  }
  StageTimer tim(POETX_STAGE_DENSE, st);
  few_dense(W, d->d_out, d->d_in, A.p, B.out(), B.ld, N, (int)B.cols, st);
}

// Block gradients are summed over exactly the call's tokens, never over padding, by kernels that follow from the descriptor: the
// order of the sum is the same in either layout and with B kept or recomputed, whichever of the tensors have padded columns.
// Only the pointers' alignment can change the kernel, which a workspace query does not see: it covers both.
size_t blockgrad_ws_bytes(const poetx_linear_desc* d) {
  const i64 N = d->n_tokens;
  size_t w = edge_blockgrad_pair_workspace_bytes(d->dtype, d->d_out, d->d_in, N, d->block);
  for (const int dim : {d->d_in, d->d_out})
    if (d->dtype == POETX_BF16 && mfma_blockgrad_preferred(dim, N, d->block)) {
      const size_t f = mfma_blockgrad_workspace_bytes(dim, N, d->block);
      if (f > w) w = f;
    }
  return align256(w);
}
// both sides' block gradients as parts, for the one-launch series backward of small blocks
size_t blockgrad_parts_bytes(const poetx_linear_desc* d, int dim) {
  return align256(edge_blockgrad_parts_bytes(d->dtype, dim, d->n_tokens, d->block));
}

// Scratch of the dense products (partials of a split contraction), both directions.  Their activation operand always lives in
// the workspace, so every plan is made for internal_columns().
size_t dense_part_bytes(const poetx_linear_desc* d) {
  const i64 N = internal_columns(d);
  const int n = d->d_out, m = d->d_in;
  const bool streams = d->dtype == POETX_BF16 && mfma_dense_supported(n, m, N);   // what is aligned; the rest is the edge kernel's
  const size_t f = few_tokens(d) ? 0 : edge_dense_workspace_bytes(d->dtype, 0, n, m, N, !streams);   // whose forward has kernels of its own
  const size_t b = edge_dense_workspace_bytes(d->dtype, 1, n, m, N, !streams);
  size_t w = f > b ? f : b;
  if (streams) {
    const size_t mf = mfma_dense_workspace_bytes(n, N, m), mb = mfma_dense_workspace_bytes(m, N, n);
    w = mf > w ? mf : w;
    w = mb > w ? mb : w;
  }
  return align256(w);
}

GradProblem grad_problem(const poetx_linear_desc* desc, const Act& U, const Act& V, int d, const int32_t* perm, float* parts = nullptr) {
  return GradProblem{U.p, V.p, U.ld, U.cols, V.ld, V.cols, desc->n_tokens, d, perm, parts};
}
bool blockgrad_streams(const poetx_linear_desc* desc, const Act& U, const Act& V, int d) {   // N in whole vectors, hence the row strides too
  return use_mfma(desc->dtype) && mfma_blockgrad_preferred(d, desc->n_tokens, desc->block) && aligned16(U.p) && aligned16(V.p);
}
void blockgrad_dispatch(const poetx_linear_desc* desc, const Act& U, const Act& V, int d, const int32_t* perm, float* dG, void* ws, hipStream_t st) {
  const int dtype = desc->dtype, b = desc->block;
  const i64 N = desc->n_tokens;
  if (blockgrad_streams(desc, U, V, d))
    mfma_blockgrad(U.p, U.ld, V.p, V.ld, d, N, perm, b, dG, ws, st);
  else if (!g_force_fma.load()) edge_blockgrad(dtype, grad_problem(desc, U, V, d, perm), b, dG, ws, st);
  else fma_blockgrad(dtype, U.p, V.p, d, N, perm, b, dG, st);
}

}  // namespace

extern "C" {

const char* poetx_status_string(int s) {
  switch (s) {
    case POETX_OK: return "ok";
    case POETX_ERR_INVALID_ARG: return "invalid argument";
    case POETX_ERR_BAD_SHAPE: return "inconsistent shapes";
    case POETX_ERR_BAD_PERM: return "not a permutation";
    case POETX_ERR_UNSUPPORTED: return "unsupported configuration";
    case POETX_ERR_WORKSPACE: return "workspace missing or too small";
    case POETX_ERR_HIP: return "HIP runtime error";
    default: return "unknown status";
  }
}

int poetx_version(void) { return 100; }

// Test hook: path != 0 forces the plain fp32-FMA kernels for every dtype.
void poetx_debug_force_fma(int on) { g_force_fma.store(on ? 1 : 0); }

size_t poetx_cnp_workspace_bytes(int32_t d, int32_t b) {
  if (d <= 0 || b <= 0) return 0;
  return align256((size_t)3 * ceil_div(d, b) * b * b * sizeof(float));  // covers both kernel families
}

int poetx_cnp_build(const float* theta, int32_t d, int32_t b, int32_t k, int32_t precision, float* G_f32,
                    void* E_bf16, void* ws, size_t ws_bytes, void* stream) {
  if (!theta || (!G_f32 && !E_bf16) || d <= 0 || b <= 0 || k < 1) return POETX_ERR_INVALID_ARG;
  if (precision != POETX_CNP_FP32 && precision != POETX_CNP_BF16) return POETX_ERR_INVALID_ARG;
  if (b > d) return POETX_ERR_BAD_SHAPE;
  if (!ws || ws_bytes < poetx_cnp_workspace_bytes(d, b)) return POETX_ERR_WORKSPACE;
  hipStream_t st = (hipStream_t)stream;
  StageTimer tm(POETX_STAGE_CNP_FWD, st);
  if (precision == POETX_CNP_BF16 && !g_force_fma.load() && mfma_cnp_supported(d, b))
    mfma_cnp_build(theta, d, b, k, G_f32, E_bf16, (float*)ws, st);
  else if (series_small(b))
    series_small_build(theta, d, b, k, G_f32, E_bf16, st);
  else
    fma_cnp_build(theta, d, b, k, G_f32, E_bf16, (float*)ws, st);
  return launch_status();
}

int poetx_cnp_build_static(const float* theta, int32_t d, int32_t b, int32_t k, int32_t precision, float* G_f32,
                           void* E_bf16, void* stream) {
  if (!theta || (!G_f32 && !E_bf16) || d <= 0 || b <= 0 || k < 1) return POETX_ERR_INVALID_ARG;
  if (precision != POETX_CNP_FP32 && precision != POETX_CNP_BF16) return POETX_ERR_INVALID_ARG;
  if (b > d) return POETX_ERR_BAD_SHAPE;
  if ((size_t)ceil_div(d, b) * b * b > kStaticCnpElems) return POETX_ERR_UNSUPPORTED;   // beyond the static scratch
  void* ws = nullptr;
  const int rc = static_scratch(&ws);
  if (rc != POETX_OK) return rc;
  // every scratch element the kernels read was written earlier in the same call: nothing to clear
  return poetx_cnp_build(theta, d, b, k, precision, G_f32, E_bf16, ws, kStaticCnpBytes, stream);
}

size_t poetx_cnp_bwd_workspace_bytes(int32_t d, int32_t b, int32_t k) {
  if (d <= 0 || b <= 0 || k < 1) return 0;
  return align256((cnp_bwd_ws_floats(ceil_div(d, b), b, k) - (size_t)ceil_div(d, b) * b * b) * sizeof(float));   // without dG itself
}

int poetx_cnp_bwd(const float* theta, const float* dG, int32_t d, int32_t b, int32_t k, int32_t precision,
                  float* dtheta, int32_t accumulate, void* ws, size_t ws_bytes, void* stream) {
  if (!theta || !dG || !dtheta || d <= 0 || b <= 0 || k < 1) return POETX_ERR_INVALID_ARG;
  if (precision != POETX_CNP_FP32 && precision != POETX_CNP_BF16) return POETX_ERR_INVALID_ARG;
  if (b > d) return POETX_ERR_BAD_SHAPE;
  if (!ws || ws_bytes < poetx_cnp_bwd_workspace_bytes(d, b, k)) return POETX_ERR_WORKSPACE;
  hipStream_t st = (hipStream_t)stream;
  StageTimer tm(POETX_STAGE_CNP_BWD, st);
  const SeriesSide side{theta, dG, 0, 1, d, dtheta};
  if (precision == POETX_CNP_BF16 && !g_force_fma.load() && mfma_cnp_supported(d, b))
    mfma_cnp_bwd(&side, 1, b, k, accumulate != 0, (float*)ws, st);
  else if (series_small(b))
    series_small_bwd(&side, 1, b, k, accumulate != 0, st);
  else
    fma_cnp_bwd(theta, dG, d, b, k, dtheta, accumulate != 0, (float*)ws, st);
  return launch_status();
}

size_t poetx_weight_q8_bytes(int32_t n, int32_t m) {
  if (n <= 0 || m <= 0) return 0;
  return weight_q8_scale_offset(n, m) + align256((size_t)n * sizeof(float));
}

int poetx_weight_quantize_q8(const void* W, int32_t dtype, int32_t n, int32_t m, void* Wq, void* stream) {
  if (!W || !Wq || n <= 0 || m <= 0 || !dtype_ok(dtype)) return POETX_ERR_INVALID_ARG;
  weight_quantize_q8_launch(dtype, W, n, m, Wq, (hipStream_t)stream);
  return launch_status();
}

int poetx_weight_dequantize_q8(const void* Wq, int32_t n, int32_t m, int32_t dtype, void* W_out, void* stream) {
  if (!Wq || !W_out || n <= 0 || m <= 0 || !dtype_ok(dtype)) return POETX_ERR_INVALID_ARG;
  weight_dequantize_q8_launch(Wq, n, m, dtype, W_out, (hipStream_t)stream);
  return launch_status();
}

int poetx_perm_blockdiag_apply_left(const void* V, void* out, int32_t d, int64_t cols, int64_t ld,
                                    const int32_t* perm, const void* blocks, int32_t b, int32_t transpose_G,
                                    int32_t dtype, void* stream) {
  if (!V || !out || !perm || !blocks || d <= 0 || cols <= 0 || b <= 0 || !dtype_ok(dtype)) return POETX_ERR_INVALID_ARG;
  if (ld < cols || b > d) return POETX_ERR_BAD_SHAPE;
  if (cols >= (1ll << 31)) return POETX_ERR_UNSUPPORTED;
  size_t bytes = (size_t)d * ld * esize(dtype);
  if (overlap(V, bytes, out, bytes)) return POETX_ERR_INVALID_ARG;
  apply_left_alone(dtype, Act{V, ld, cols}, Act{out, ld, cols}, d, perm, blocks, b, transpose_G != 0, (hipStream_t)stream);
  return launch_status();
}

int poetx_perm_blockdiag_apply_right(const void* V, void* out, int64_t rows, int32_t d, int64_t ld,
                                     const int32_t* perm, const void* blocks, int32_t b, int32_t transpose_G,
                                     int32_t dtype, void* stream) {
  if (!V || !out || !perm || !blocks || d <= 0 || rows <= 0 || b <= 0 || !dtype_ok(dtype)) return POETX_ERR_INVALID_ARG;
  if (ld < d || b > d) return POETX_ERR_BAD_SHAPE;
  if (rows >= (1ll << 31)) return POETX_ERR_UNSUPPORTED;
  size_t bytes = (size_t)rows * ld * esize(dtype);
  if (overlap(V, bytes, out, bytes)) return POETX_ERR_INVALID_ARG;
  StageTimer tm(POETX_STAGE_APPLY, (hipStream_t)stream);
  fma_apply_right(dtype, V, out, rows, d, ld, perm, blocks, b, transpose_G != 0, (hipStream_t)stream);
  return launch_status();
}

size_t poetx_merge_workspace_bytes(int32_t n, int32_t m, int32_t dtype) {
  if (n <= 0 || m <= 0 || !dtype_ok(dtype)) return 0;
  return 2 * align256((size_t)n * m * esize(dtype));
}

int poetx_merge_weight(const void* W, void* W_out, int32_t n, int32_t m, const int32_t* perm_R, const int32_t* perm_P,
                       const void* blocks_R, const void* blocks_P, int32_t b, int32_t dtype, void* ws, size_t ws_bytes,
                       void* stream) {
  if (!W || !W_out || !perm_R || !perm_P || !blocks_R || !blocks_P || n <= 0 || m <= 0 || b <= 0 || !dtype_ok(dtype))
    return POETX_ERR_INVALID_ARG;
  if (b > n || b > m) return POETX_ERR_BAD_SHAPE;
  const size_t bytes = (size_t)n * m * esize(dtype);
  if (overlap(W, bytes, W_out, bytes)) return POETX_ERR_INVALID_ARG;
  if (!ws || ws_bytes < poetx_merge_workspace_bytes(n, m, dtype)) return POETX_ERR_WORKSPACE;
  hipStream_t st = (hipStream_t)stream;
  void* T1 = ws;
  void* T2 = (char*)ws + align256(bytes);
  // W (n x m) is feature major for the output side (rows = output features): P^T W is a left apply.
  // The input side acts on the columns; a column gather is a row gather of the transpose, so the
  // product with R^T runs as R (P^T W)^T on the transposed matrix and is transposed back.
  apply_left_alone(dtype, Act{W, m, m}, Act{T1, m, m}, n, perm_P, blocks_P, b, 1, st);        // T1 = P^T W         (n x m)
  {
    StageTimer tm(POETX_STAGE_LAYOUT, st);
    transpose_launch(dtype, T1, T2, n, m, m, n, n, st);                                   // T2 = T1^T          (m x n)
  }
  apply_left_alone(dtype, Act{T2, n, n}, Act{T1, n, n}, m, perm_R, blocks_R, b, 0, st);       // T1 = R T2          (m x n)
  {
    StageTimer tm(POETX_STAGE_LAYOUT, st);
    transpose_launch(dtype, T1, W_out, m, n, n, m, m, st);                                // W_out = (R T2)^T = P^T W R^T
  }
  return launch_status();
}

int poetx_perm_validate(const int32_t* perm, int32_t d, int32_t* scratch, void* stream) {
  if (!perm || !scratch || d <= 0) return POETX_ERR_INVALID_ARG;
  hipStream_t st = (hipStream_t)stream;
  perm_validate_launch(perm, d, scratch, st);
  int32_t bad = 0;
  if (hipMemcpyAsync(&bad, scratch + d, sizeof(int32_t), hipMemcpyDeviceToHost, st) != hipSuccess) return POETX_ERR_HIP;
  if (hipStreamSynchronize(st) != hipSuccess) return POETX_ERR_HIP;
  return bad ? POETX_ERR_BAD_PERM : POETX_OK;
}

static size_t dequantised_weight_bytes(const poetx_linear_desc* desc) {
  return ((desc->flags & POETX_FLAG_W_INT8) && !weight_in_kernel(desc))
             ? align256((size_t)desc->d_out * desc->d_in * esize(desc->dtype)) : 0;
}

// The weight the dense product reads: W itself, or its dequantised copy made at `scratch`.
static const void* resolve_weight(const poetx_linear_desc* desc, const void* W, void* scratch, hipStream_t st) {
  if (!(desc->flags & POETX_FLAG_W_INT8) || weight_in_kernel(desc)) return W;
  StageTimer tm(POETX_STAGE_DEQUANT, st);
  weight_dequantize_q8_launch(W, desc->d_out, desc->d_in, desc->dtype, scratch, st);
  return scratch;
}

// Bytes of a workspace activation of `rows` features.
static size_t act_bytes(const poetx_linear_desc* d, int rows) {
  return align256((size_t)rows * (size_t)internal_columns(d) * esize(d->dtype));
}

// Token-major callers: feature-major copies of the call's activations (at most X, dZ / Z and dX)
// live behind the regular workspace.
static size_t layout_staging_bytes(const poetx_linear_desc* d) {
  if (d->layout != POETX_TOKEN_MAJOR) return 0;
  return 2 * act_bytes(d, d->d_in) + act_bytes(d, d->d_out);
}
static size_t core_workspace_bytes(const poetx_linear_desc* desc);

size_t poetx_linear_workspace_bytes(const poetx_linear_desc* desc) {
  if (check_desc(desc) != POETX_OK) return 0;
  return core_workspace_bytes(desc) + layout_staging_bytes(desc);
}

int poetx_linear_path(const poetx_linear_desc* d) {
  const int rc = check_desc(d);
  if (rc) return -rc;
  const int m = d->d_in, n = d->d_out, b = d->block;
  const i64 N = d->n_tokens, Ni = internal_columns(d);
  int path = 0;
  // each bit by what the dispatch asks; the other stages of fp32 tensors take the edge-handling kernels
  if (d->dtype == POETX_F32 && !g_force_fma.load() && mfma_dense_f32_preferred(n, m, n, N) && mfma_dense_f32_preferred(n, m, m, N)) path |= POETX_PATH_DENSE;
  if (!use_mfma(d->dtype)) return path;
  if (apply_streams(d, m) && apply_streams(d, n)) path |= POETX_PATH_APPLY;
  if (mfma_dense_supported(n, m, Ni)) path |= POETX_PATH_DENSE;
  if (mfma_blockgrad_preferred(m, N, b) && mfma_blockgrad_preferred(n, N, b)) path |= POETX_PATH_BLOCKGRAD;
  if (d->cnp_precision == POETX_CNP_BF16 && mfma_cnp_supported(m, b) && mfma_cnp_supported(n, b)) {
    path |= POETX_PATH_SERIES;
    if (lds_cnp_supported(m, b) && lds_cnp_supported(n, b)) path |= POETX_PATH_SERIES_ON_CHIP;
    if (bwd_one_pass(d)) path |= POETX_PATH_BWD_ONE_PASS;
  }
  if (weight_in_kernel(d)) path |= POETX_PATH_W_INT8_IN_KERNEL;
  return path;
}

// Feature-major <-> token-major copies around a call.  in(): the feature-major form of an input -- the caller's tensor
// itself, or its transposed copy in the workspace (padded like every workspace activation); out(): where the call
// should write a feature-major output; finish(): transposes the registered outputs into the caller's token-major
// buffers.
class LayoutStaging {
 public:
  LayoutStaging(const poetx_linear_desc* d, void* ws, hipStream_t st)
      : d_(d), on_(d->layout == POETX_TOKEN_MAJOR), dt_(d->dtype), N_(d->n_tokens), Ni_(internal_columns(d)), st_(st),
        next_(on_ ? (char*)ws + core_workspace_bytes(d) : nullptr), n_out_(0) {}
  Act in(const void* p, int rows) {
    if (!on_ || !p) return Act{p, N_, N_};
    void* t = take(rows);
    StageTimer tm(POETX_STAGE_LAYOUT, st_);
    transpose_launch(dt_, p, t, N_, rows, rows, Ni_, Ni_, st_);        // [N][rows] -> [rows][Ni], zeros past N
    return Act{t, Ni_, Ni_};
  }
  Act out(void* p, int rows) {
    if (!on_ || !p) return Act{p, N_, N_};
    void* t = take(rows);
    outs_[n_out_].user = p; outs_[n_out_].tmp = t; outs_[n_out_].rows = rows; ++n_out_;
    return Act{t, Ni_, Ni_};
  }
  void finish() {
    for (int i = 0; i < n_out_; ++i) {
      StageTimer tm(POETX_STAGE_LAYOUT, st_);
      transpose_launch(dt_, outs_[i].tmp, outs_[i].user, outs_[i].rows, N_, Ni_, outs_[i].rows, outs_[i].rows, st_);   // [rows][N] -> [N][rows]
    }
  }
 private:
  void* take(int rows) {
    void* t = next_;
    next_ += act_bytes(d_, rows);
    return t;
  }
  const poetx_linear_desc* d_;
  bool on_; int dt_; i64 N_, Ni_; hipStream_t st_; char* next_;
  struct { void* user; void* tmp; int rows; } outs_[2];
  int n_out_;
};

// poetx_linear_bwd called without saved_B recomputes B itself: B, then the dequantised weight (kept for both
// of the call's dense products), sit at the very end of the workspace.
static size_t recompute_tail_bytes(const poetx_linear_desc* desc) {
  if (!(desc->flags & POETX_FLAG_RECOMPUTE_B)) return 0;
  return act_bytes(desc, desc->d_out) + dequantised_weight_bytes(desc);
}

static size_t core_workspace_bytes(const poetx_linear_desc* desc) {
  const i64 Ni = internal_columns(desc);
  const size_t actm = act_bytes(desc, desc->d_in), actn = act_bytes(desc, desc->d_out);
  size_t fwd = actm;                                    // A = R^T X
  if (desc->flags & POETX_FLAG_RECOMPUTE_B) fwd += actn;  // B lives here too
  const size_t wdeq = dequantised_weight_bytes(desc);   // only where no kernel converts on the fly
  fwd += wdeq;                                          // dequantised weight behind A (and B), then the dense product's partials
  size_t bwi = actn + wdeq;                             // dB = P dZ; partials likewise
  const size_t bg = blockgrad_ws_bytes(desc);
  const size_t chain = cnp_bwd_ws_floats(desc);
  size_t skew = align256(chain * sizeof(float)) + bg;
  if (series_small_supported(desc->block)) {
    const size_t parts = blockgrad_parts_bytes(desc, desc->d_in) + blockgrad_parts_bytes(desc, desc->d_out);
    if (parts > skew) skew = parts;
  }
  // A few tokens' partials (of the backward product alone: up to sixteen ranges, or 1024 tiles of 32 x 32) mostly disappear in what the series needs, and the price of its plan,
  // which this query of every call then leaves out, is most of its time.
  const size_t few = 64 * (size_t)desc->d_in * (size_t)Ni, most = few > (4u << 20) ? few : 4u << 20;
  const size_t part = few_tokens(desc) && bwi + most <= skew ? 0 : dense_part_bytes(desc);
  fwd += part;
  bwi += part;
  size_t w = fwd > bwi ? fwd : bwi;
  if (skew > w) w = skew;
  // poetx_linear_bwd keeps dA (and, on its one-pass path, dB) in the workspace next to what the two
  // halves need: dA | two-call scratch, or dA | dB | dG + chain | partials or dequantised weight
  const size_t two_calls = bwi > skew ? bwi : skew;
  size_t bwd = actm + two_calls;
  const i64 N = desc->n_tokens;
  if (desc->dtype == POETX_BF16 && Ni == N && mfma_apply_grad_supported(desc->d_in, N, N, desc->block) &&
      mfma_apply_grad_supported(desc->d_out, N, N, desc->block)) {
    size_t tail = align256(mfma_apply_grad_workspace_bytes(desc->d_in, N));
    const size_t po = align256(mfma_apply_grad_workspace_bytes(desc->d_out, N));
    if (po > tail) tail = po;
    if (wdeq + part > tail) tail = wdeq + part;
    const size_t one_pass = actm + actn + align256(chain * sizeof(float)) + tail;
    if (one_pass > bwd) bwd = one_pass;
  }
  bwd += recompute_tail_bytes(desc);
  return w > bwd ? w : bwd;
}

int poetx_linear_fwd(const poetx_linear_desc* desc, const void* X, const void* W, const int32_t* perm_R,
                     const int32_t* perm_P, const void* blocks_R, const void* blocks_P, void* Z, void* saved_B,
                     void* ws, size_t ws_bytes, void* stream) {
  int rc = check_desc(desc);
  if (rc) return rc;
  if (!X || !W || !perm_R || !perm_P || !blocks_R || !blocks_P || !Z) return POETX_ERR_INVALID_ARG;
  if (!saved_B && !(desc->flags & POETX_FLAG_RECOMPUTE_B)) return POETX_ERR_INVALID_ARG;
  if (!ws || ws_bytes < poetx_linear_workspace_bytes(desc)) return POETX_ERR_WORKSPACE;
  hipStream_t st = (hipStream_t)stream;
  const int m = desc->d_in, n = desc->d_out, b = desc->block, dt = desc->dtype;
  const i64 N = desc->n_tokens, Ni = internal_columns(desc);
  const Act A{ws, Ni, Ni};
  char* after = (char*)ws + act_bytes(desc, m);
  Act B{saved_B, N, N};
  if (!saved_B) {  // memory-saving variant: scratch only
    B = Act{after, Ni, Ni};
    after += act_bytes(desc, n);
  }
  W = resolve_weight(desc, W, after, st);
  void* part = after + dequantised_weight_bytes(desc);
  if (few_tokens(desc)) {
    few_b(desc, X, W, perm_R, blocks_R, A, B, st);
    StageTimer tm(POETX_STAGE_APPLY, st);
    const bool tok = desc->layout == POETX_TOKEN_MAJOR;
    few_apply(B.p, B.ld, false, Z, tok ? n : N, tok, n, (int)N, perm_P, blocks_P, b, 1, st);
    return launch_status();
  }
  if (reads_tokens_in_place(desc)) {
    {
      StageTimer tm(POETX_STAGE_APPLY, st);
      edge_apply_tokens(dt, X, m, true, A.out(), Ni, false, m, N, Ni, perm_R, blocks_R, b, 1, st);
    }
    dense_dispatch(desc, 0, W, A, B, part, st, weight_in_kernel(desc));
    StageTimer tm(POETX_STAGE_APPLY, st);
    edge_apply_tokens(dt, B.p, B.ld, false, Z, n, true, n, N, N, perm_P, blocks_P, b, 1, st);
    return launch_status();
  }
  LayoutStaging lay(desc, ws, st);
  const Act x = lay.in(X, m), z = lay.out(Z, n);
  apply_left(desc, x, A, m, perm_R, blocks_R, 1, st);              // mm1: A = R^T X
  dense_dispatch(desc, 0, W, A, B, part, st, weight_in_kernel(desc));    // mm2: B = W A
  apply_left(desc, B, z, n, perm_P, blocks_P, 1, st);              // mm3: Z = P^T B
  lay.finish();
  return launch_status();
}

int poetx_linear_recompute_b(const poetx_linear_desc* desc, const void* X, const void* W, const int32_t* perm_R,
                             const void* blocks_R, void* B_out, void* ws, size_t ws_bytes, void* stream) {
  int rc = check_desc(desc);
  if (rc) return rc;
  if (!X || !W || !perm_R || !blocks_R || !B_out) return POETX_ERR_INVALID_ARG;
  if (!ws || ws_bytes < poetx_linear_workspace_bytes(desc)) return POETX_ERR_WORKSPACE;
  hipStream_t st = (hipStream_t)stream;
  const int m = desc->d_in;
  const i64 N = desc->n_tokens, Ni = internal_columns(desc);
  const Act A{ws, Ni, Ni};
  char* after = (char*)ws + act_bytes(desc, m);
  W = resolve_weight(desc, W, after, st);
  if (few_tokens(desc)) {
    few_b(desc, X, W, perm_R, blocks_R, A, Act{B_out, N, N}, st);
    return launch_status();
  }
  LayoutStaging lay(desc, ws, st);
  const Act x = lay.in(X, m);
  apply_left(desc, x, A, m, perm_R, blocks_R, 1, st);  // A = R^T X
  dense_dispatch(desc, 0, W, A, Act{B_out, N, N}, after + dequantised_weight_bytes(desc), st, weight_in_kernel(desc));   // B = W A
  return launch_status();
}

// dX = R dA beside the block gradients of a one-call backward (small blocks): what bwd_input_impl leaves out and bwd_skew_impl then does
struct JoinedApply {
  const void* blocks_R;
  Act dX;
};
static bool joins_apply(const poetx_linear_desc* d) {
  const int m = d->d_in, n = d->d_out, b = d->block;
  return !(d->flags & POETX_FLAG_BLOCK_GRADS) && series_small(b) && !apply_streams(d, m) && !fma_apply_left_preferred(m, d->n_tokens, b) &&
         edge_apply_joins_blockgrads(d->dtype, m, d->n_tokens, n, m, d->n_tokens, b);
}

// dB = P dZ, dA = W^T dB, dX = R dA (unless it is joined); ws holds dB (and the dequantised weight behind it)
static void bwd_input_impl(const poetx_linear_desc* desc, const Act& dZ, const void* W, const int32_t* perm_R,
                           const int32_t* perm_P, const void* blocks_R, const void* blocks_P, const Act& dX, const Act& dA,
                           void* ws, hipStream_t st, const void* W_resolved = nullptr, bool joined = false) {
  const int m = desc->d_in, n = desc->d_out;
  const i64 Ni = internal_columns(desc);
  const Act dB{ws, Ni, Ni};
  char* after = (char*)ws + act_bytes(desc, n);
  W = W_resolved ? W_resolved : resolve_weight(desc, W, after, st);
  apply_left(desc, dZ, dB, n, perm_P, blocks_P, 0, st);  // dB = P dZ
  dense_dispatch(desc, 1, W, dB, dA, after + dequantised_weight_bytes(desc), st, weight_in_kernel(desc));   // dA = W^T dB
  if (!joined) apply_left(desc, dA, dX, m, perm_R, blocks_R, 0, st);  // dX = R dA
}

int poetx_linear_bwd_input(const poetx_linear_desc* desc, const void* dZ, const void* W, const int32_t* perm_R,
                           const int32_t* perm_P, const void* blocks_R, const void* blocks_P, void* dX, void* dA,
                           void* ws, size_t ws_bytes, void* stream) {
  int rc = check_desc(desc);
  if (rc) return rc;
  if (!dZ || !W || !perm_R || !perm_P || !blocks_R || !blocks_P || !dX || !dA) return POETX_ERR_INVALID_ARG;
  if (!ws || ws_bytes < poetx_linear_workspace_bytes(desc)) return POETX_ERR_WORKSPACE;
  LayoutStaging lay(desc, ws, (hipStream_t)stream);
  const Act dz = lay.in(dZ, desc->d_out), dx = lay.out(dX, desc->d_in);
  bwd_input_impl(desc, dz, W, perm_R, perm_P, blocks_R, blocks_P, dx, Act{dA, desc->n_tokens, desc->n_tokens}, ws, (hipStream_t)stream);
  lay.finish();
  return launch_status();
}

// Series backward of both sides as one batch (a side alone leaves most CUs empty): dG holds the block gradients of the
// P side, then of the R side; the chain's scratch follows.
static void cnp_bwd_both(const float* theta_R, const float* theta_P, float* dG, int m, int n, int b, int k,
                         float* dtheta_R, float* dtheta_P, int accumulate, hipStream_t st) {
  const int nbP = n / b, nbt = nbP + m / b;
  const size_t bb = (size_t)b * b;
  const SeriesSide sides[2] = {{theta_P, dG, 0, 1, n, dtheta_P}, {theta_R, dG + nbP * bb, 0, 1, m, dtheta_R}};
  StageTimer tm(POETX_STAGE_CNP_BWD, st);
  mfma_cnp_bwd(sides, 2, b, k, accumulate != 0, dG + nbt * bb, st);
}

static void bwd_skew_impl(const poetx_linear_desc* desc, const Act& X, const Act& dZ, const Act& saved_B,
                          const Act& dA, const int32_t* perm_R, const int32_t* perm_P, const float* theta_R,
                          const float* theta_P, float* dtheta_R, float* dtheta_P, int32_t accumulate, void* ws,
                          hipStream_t st, const JoinedApply* joined = nullptr) {
  const int m = desc->d_in, n = desc->d_out, b = desc->block, dt = desc->dtype, k = desc->neumann_k;
  const int dmax = m > n ? m : n;
  void* bg_ws = (char*)ws + align256(cnp_bwd_ws_floats(desc) * sizeof(float));
  // POETX_FLAG_BLOCK_GRADS: the block gradients go to the caller (in place of dtheta) and the series
  // backward is left to poetx_cnp_bwd
  const bool defer = (desc->flags & POETX_FLAG_BLOCK_GRADS) != 0;
  if (desc->cnp_precision == POETX_CNP_BF16 && !g_force_fma.load() && use_mfma(dt) && mfma_cnp_supported(m, b) &&
      mfma_cnp_supported(n, b)) {
    // Both sides' blocks go through the series backward as one batch (P side first): the chains
    // are latency bound and a side alone leaves most CUs empty.
    const int nbP = n / b;
    const size_t bb = (size_t)b * b;
    float* dG = (float*)ws;                                   // [nbt][b][b]
    {
      StageTimer tm(POETX_STAGE_BLOCKGRAD, st);
      float *dG_P = defer ? dtheta_P : dG, *dG_R = defer ? dtheta_R : dG + nbP * bb;   // B' dZ'^T, X' dA'^T
      if (blockgrad_streams(desc, saved_B, dZ, n) || blockgrad_streams(desc, X, dA, m)) {
        blockgrad_dispatch(desc, saved_B, dZ, n, perm_P, dG_P, bg_ws, st);
        blockgrad_dispatch(desc, X, dA, m, perm_R, dG_R, bg_ws, st);
      } else {
        edge_blockgrad_pair(dt, grad_problem(desc, saved_B, dZ, n, perm_P), grad_problem(desc, X, dA, m, perm_R), b, dG_P, dG_R, bg_ws, st);
      }
    }
    if (defer) return;
    cnp_bwd_both(theta_R, theta_P, dG, m, n, b, k, dtheta_R, dtheta_P, accumulate, st);
    return;
  }
  if (!defer && series_small(b)) {
    // Both sides' block gradients, still split over token ranges, then one launch that adds the parts, runs the
    // series backward and projects.  The P side's parts sit where the other paths keep dG and the chain.
    SeriesSide sides[2] = {{theta_P, (const float*)ws, (i64)ceil_div(n, b) * b * b, 1, n, dtheta_P},
                           {theta_R, (const float*)((char*)ws + blockgrad_parts_bytes(desc, n)), (i64)ceil_div(m, b) * b * b, 1, m, dtheta_R}};
    {
      StageTimer tm(POETX_STAGE_BLOCKGRAD, st);
      const GradProblem gp = grad_problem(desc, saved_B, dZ, n, perm_P, (float*)sides[0].dG), gr = grad_problem(desc, X, dA, m, perm_R, (float*)sides[1].dG);
      if (joined)
        edge_apply_blockgrad_parts(dt, dA.p, dA.ld, joined->dX.out(), joined->dX.ld, min64(dA.cols, joined->dX.cols), joined->dX.cols, desc->n_tokens, joined->blocks_R, gp, gr, b,
                                   &sides[0].nsplit, &sides[1].nsplit, st);
      else
        edge_blockgrad_parts_pair(dt, gp, gr, b, &sides[0].nsplit, &sides[1].nsplit, st);
    }
    StageTimer tm(POETX_STAGE_CNP_BWD, st);
    series_small_bwd(sides, 2, b, k, accumulate != 0, st);
    return;
  }
  float* dG = (float*)ws;
  float* chain = dG + (size_t)ceil_div(dmax, b) * b * b;
  for (int side = 0; side < 2; ++side) {
    const Act& U = side == 0 ? saved_B : X;   // mm3 backward: dG_P = B' dZ'^T; mm1 backward: dG_R = X' dA'^T
    const Act& V = side == 0 ? dZ : dA;
    const int d = side == 0 ? n : m;
    const int32_t* perm = side == 0 ? perm_P : perm_R;
    const float* theta = side == 0 ? theta_P : theta_R;
    float* dtheta = side == 0 ? dtheta_P : dtheta_R;
    const bool fast_cnp = desc->cnp_precision == POETX_CNP_BF16 && !g_force_fma.load() && mfma_cnp_supported(d, b);
    float* dGs = defer ? dtheta : dG;
    {
      StageTimer tm(POETX_STAGE_BLOCKGRAD, st);
      blockgrad_dispatch(desc, U, V, d, perm, dGs, bg_ws, st);
    }
    if (!defer) {
      StageTimer tm(POETX_STAGE_CNP_BWD, st);
      const SeriesSide one{theta, dG, 0, 1, d, dtheta};
      if (fast_cnp) mfma_cnp_bwd(&one, 1, b, k, accumulate != 0, chain, st);
      else fma_cnp_bwd(theta, dG, d, b, k, dtheta, accumulate != 0, chain, st);
    }
  }
}

int poetx_linear_bwd_skew(const poetx_linear_desc* desc, const void* X, const void* dZ, const void* saved_B,
                          const void* dA, const int32_t* perm_R, const int32_t* perm_P, const float* theta_R,
                          const float* theta_P, float* dtheta_R, float* dtheta_P, int32_t accumulate, void* ws,
                          size_t ws_bytes, void* stream) {
  int rc = check_desc(desc);
  if (rc) return rc;
  if (!X || !dZ || !saved_B || !dA || !perm_R || !perm_P || !theta_R || !theta_P || !dtheta_R || !dtheta_P)
    return POETX_ERR_INVALID_ARG;
  if (!ws || ws_bytes < poetx_linear_workspace_bytes(desc)) return POETX_ERR_WORKSPACE;
  LayoutStaging lay(desc, ws, (hipStream_t)stream);
  const i64 N = desc->n_tokens;
  const Act x = lay.in(X, desc->d_in), dz = lay.in(dZ, desc->d_out);
  bwd_skew_impl(desc, x, dz, Act{saved_B, N, N}, Act{dA, N, N}, perm_R, perm_P, theta_R, theta_P, dtheta_R, dtheta_P, accumulate, ws,
                (hipStream_t)stream);
  return launch_status();
}

int poetx_linear_bwd(const poetx_linear_desc* desc, const void* X, const void* dZ, const void* saved_B, const void* W,
                     const int32_t* perm_R, const int32_t* perm_P, const void* blocks_R, const void* blocks_P,
                     const float* theta_R, const float* theta_P, void* dX, float* dtheta_R, float* dtheta_P,
                     int32_t accumulate, void* ws, size_t ws_bytes, void* stream) {
  int rc = check_desc(desc);
  if (rc) return rc;
  if (!X || !dZ || !W || !perm_R || !perm_P || !blocks_R || !blocks_P || !theta_R || !theta_P || !dX ||
      !dtheta_R || !dtheta_P)
    return POETX_ERR_INVALID_ARG;
  if (!saved_B && !(desc->flags & POETX_FLAG_RECOMPUTE_B)) return POETX_ERR_INVALID_ARG;
  if (!ws || ws_bytes < poetx_linear_workspace_bytes(desc)) return POETX_ERR_WORKSPACE;
  hipStream_t st = (hipStream_t)stream;
  const int m = desc->d_in, n = desc->d_out, b = desc->block, k = desc->neumann_k;
  const i64 N = desc->n_tokens, Ni = internal_columns(desc);
  LayoutStaging lay(desc, ws, st);
  const Act x = lay.in(X, m), dz = lay.in(dZ, n), dx = lay.out(dX, m);
  const Act dA{ws, Ni, Ni};                                        // lives until the R side is done
  char* rest = (char*)ws + act_bytes(desc, m);
  const void* W_resolved = nullptr;
  Act B{saved_B, N, N};
  if (!saved_B) {
    // Gradient checkpoint inside the call (Sec. 3.5, memory-saving variant): A = R^T X goes where dA will
    // be, B = W A to the end of the workspace; a quantised weight is dequantised once for both products.
    char* end = (char*)ws + core_workspace_bytes(desc);
    char* w_keep = end - dequantised_weight_bytes(desc);
    B = Act{w_keep - act_bytes(desc, n), Ni, Ni};
    W_resolved = resolve_weight(desc, W, w_keep, st);
    if (few_tokens(desc)) {
      few_b(desc, X, W_resolved, perm_R, blocks_R, dA, B, st);
    } else {
      apply_left(desc, x, dA, m, perm_R, blocks_R, 1, st);
      dense_dispatch(desc, 0, W_resolved, dA, B, rest, st, weight_in_kernel(desc));   // partials where dB will be
    }
  }
  // Each side's gradient is streamed once where the call's tokens are whole tiles: dB = P dZ together with
  // dG_P = B' dZ'^T, then dA = W^T dB, then dX = R dA together with dG_R = X' dA'^T (Sec. 3.5).  A token count that is padded
  // in the workspace goes through the two halves: the caller's own tensors have no padded columns to stream.
  const Act dB{rest, Ni, Ni};
  const bool one_pass = bwd_one_pass(desc) && aligned16(dz.p) && aligned16(B.p) && aligned16(x.p) && aligned16(dx.p) && aligned16(blocks_R) &&
                        aligned16(blocks_P);
  if (!one_pass) {   // the same values through the two halves
    const JoinedApply join{blocks_R, dx};
    const bool joined = joins_apply(desc);
    bwd_input_impl(desc, dz, W, perm_R, perm_P, blocks_R, blocks_P, dx, dA, rest, st, W_resolved, joined);
    bwd_skew_impl(desc, x, dz, B, dA, perm_R, perm_P, theta_R, theta_P, dtheta_R, dtheta_P, accumulate, rest, st, joined ? &join : nullptr);
    lay.finish();
    return launch_status();
  }
  char* after_dB = rest + act_bytes(desc, n);
  const int nbP = n / b;
  const size_t bb = (size_t)b * b;
  float* dG = (float*)after_dB;                                    // both sides' block gradients, then chain scratch
  void* part = after_dB + align256(cnp_bwd_ws_floats(desc) * sizeof(float));
  const bool defer = (desc->flags & POETX_FLAG_BLOCK_GRADS) != 0;   // block gradients to the caller, no series backward
  float* dG_P = defer ? dtheta_P : dG;
  float* dG_R = defer ? dtheta_R : dG + nbP * bb;
  auto side = [&](const Act& V, const Act& U, const Act& out, int d, const int32_t* perm, const void* blocks, float* dGs) {
    StageTimer tm(POETX_STAGE_APPLY_GRAD, st);
    mfma_apply_grad(V.p, U.p, out.out(), d, N, N, perm, blocks, 0, dGs, part, st);
  };
  side(dz, B, dB, n, perm_P, blocks_P, dG_P);
  W = W_resolved ? W_resolved : resolve_weight(desc, W, part, st);   // the P side's partials are reduced by now (stream order): same space
  dense_dispatch(desc, 1, W, dB, dA, (char*)part + dequantised_weight_bytes(desc), st, weight_in_kernel(desc));
  side(dA, x, dx, m, perm_R, blocks_R, dG_R);
  lay.finish();
  if (defer) return launch_status();
  cnp_bwd_both(theta_R, theta_P, dG, m, n, b, k, dtheta_R, dtheta_P, accumulate, st);
  return launch_status();
}

}  // extern "C"
