// Dense bf16 products of the POET-X linear layer on the matrix cores (mfma_dense_kernel.h): which tile and split a product takes, and its launches.
// Products of too few such tiles for the chip take 256 x 128 or 128 x 128 ones, or split their contraction (see pick_plan).
#include "edge_gemm.h"
#include "mfma_dense_kernel.h"

namespace poetx {
namespace {

using namespace dense;

int compute_units() {
  static const int n = [] {
    int dev = 0, cu = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cu <= 0)
      cu = 256;
    return cu;
  }();
  return n;
}

// out (M x N bf16, row stride ld_out, any alignment) = sum of the parts [split][M][Np], in order; eight columns per thread
__global__ __launch_bounds__(256) void dense_reduce_kernel(const float* __restrict__ parts, int splits, i64 M, i64 Np, uint16_t* __restrict__ out,
                                                           i64 ld_out, int N) {
  const i64 idx = (i64)blockIdx.x * 256 + threadIdx.x, row = idx / (Np / 8);
  const int col = (int)(idx - row * (Np / 8)) * 8;
  if (row >= M || col >= N) return;
  float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  const float* p = parts + row * Np + col;
  for (int z = 0; z < splits; ++z, p += M * Np) {
    const float4 lo = *reinterpret_cast<const float4*>(p), hi = *reinterpret_cast<const float4*>(p + 4);
    v[0] += lo.x; v[1] += lo.y; v[2] += lo.z; v[3] += lo.w;
    v[4] += hi.x; v[5] += hi.y; v[6] += hi.z; v[7] += hi.w;
  }
  edge::store8(out + row * ld_out + col, v, N - col);
}

template <bool A_KMAJOR, Out OUT, class C>
void launch_tile(DenseArgs g, i64 M, i64 N, hipStream_t st) {
  auto kern = dense_stream_kernel<A_KMAJOR, OUT, 0, C>;
  static const bool configured =
      hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS_BYTES) == hipSuccess;
  (void)configured;
  g.tiles_m = (int)(M / C::BM);
  g.tiles_n = (int)(N / C::BN);
  const int T = g.tiles_m * g.tiles_n * g.splits, cus = compute_units();
  hipLaunchKernelGGL(kern, dim3(T < cus || g.longer > 0 ? T : cus), dim3(256), C::LDS_BYTES, st, g);
}

// ---- which tile, how many contraction ranges ----------------------------------------------------
// Estimated time: rounds of the chip, times a tile's time, times the depth.  Measured per 4096 of depth with the whole chip
// busy: 94 us for a 256 x 256 tile, 0.65 of that for 256 x 128 and 0.39 for 128 x 128 (half and a quarter of the work: smaller
// tiles move more operand bytes per flop), so a smaller tile pays where it takes the place of idle CUs (4096 x 4096 x 2048, 128
// large tiles: 90 -> 73 us on 256 x 128; 2048 x 2048 x 2048, 64: 44 -> 26 us on 128 x 128; both with the 32 x 32 x 16 kernel).  Splitting the contraction of the
// smallest tile adds fp32 parts written and read at about 4 TB/s and a launch (5 us).  A range is a whole number of pairs of stages; where that
// leaves them unequal, a workgroup has one, hence no more than 256 of them (forward calls, four equal ranges / eight of 34 and 36 stages, us: 256 x 8960, 512 tokens 41.4 / 36.0; of 40 and 42, 512 x 10496, 256
// 41.0 / 35.5).
enum { T256 = 0, T256x128 = 1, T128 = 2 };
struct DensePlan {
  int tile, splits;
};
DensePlan pick_plan(i64 M, i64 N, i64 K) {
  const double cost[3] = {1.0, 0.65, 0.39};
  const int bm[3] = {256, 256, 128}, bn[3] = {256, 128, 128};
  DensePlan best{T256, 1};
  double best_us = 0.0;
  for (int t = 0; t < 3; ++t)
    for (int s = 1; s <= (t == T128 ? 16 : 1); s *= 2) {
      if ((K / BK) % s != 0 || K / s < 256) break;
      const double units = (double)(M / bm[t]) * (double)(N / bn[t]) * s;
      const ContractionRange range = contraction_ranges((int)(K / BK), s);
      if (range.longer > 0 && units > 256) break;
      const double rounds = (double)(long long)((units + 255) / 256);
      double us = rounds * cost[t] * 94.0 / 4096.0 * (double)((range.ktiles + (range.longer > 0 ? 2 : 0)) * BK);
      if (s > 1) us += 8.0 * s * (double)M * (double)N / 4e6 + 5.0;
      if (best_us == 0.0 || us < 0.97 * best_us) { best_us = us; best = DensePlan{t, s}; }
    }
  return best;
}

template <bool A_KMAJOR, Out OUT>
void launch_dense(const DenseArgs& g, int tile, i64 M, i64 N, hipStream_t st) {
  switch (tile) {
    case T128: launch_tile<A_KMAJOR, OUT, Tile128>(g, M, N, st); break;
    case T256x128: launch_tile<A_KMAJOR, OUT, Tile256x128>(g, M, N, st); break;
    default: launch_tile<A_KMAJOR, OUT, Tile256>(g, M, N, st); break;
  }
}

}  // namespace

bool mfma_dense_supported(int n, int m, i64 N) {
  // per-lane load offsets are 32-bit: 255 rows of the wider operand must stay below 4 GB
  return n % 256 == 0 && m % 256 == 0 && N % 256 == 0 && N < (1ll << 22) && (i64)(n > m ? n : m) < (1ll << 22);
}

// Padding costs up to 255 tokens of work and, for token-major callers, longer transposes; it buys a kernel two to four times
// as fast as the edge one once there is enough of it.  Whole forward passes, edge against padded, us: 2048 x 2048 with 40
// tokens 21 / 26, 70: 36 / 31, 300: 48 / 35, 1500: 81 / 40; 1024 x 1024 with 600: 28 / 28, 1000: 33 / 29; 4096 x 14336 with
// 40: 73 / 53, 70: 208 / 59, 300: 383 / 91.
bool mfma_dense_worth_padding(int n, int m, i64 N) { return N > 64 && (i64)n * m * ((N + 255) / 256 * 256) >= (1ll << 30); }

size_t mfma_dense_workspace_bytes(i64 M, i64 N, i64 K) {
  const DensePlan p = pick_plan(M, N, K);
  return p.splits > 1 ? (size_t)p.splits * M * N * sizeof(float) : 0;
}

int mfma_dense_splits(i64 M, i64 N, i64 K) { return pick_plan(M, N, K).splits; }

void mfma_dense_reduce(const float* parts, int splits, i64 M, i64 Np, void* out, i64 ld_out, i64 N, hipStream_t st) {
  hipLaunchKernelGGL(dense_reduce_kernel, dim3((unsigned)((M * (Np / 8) + 255) / 256)), dim3(256), 0, st, parts, splits, M, Np, (uint16_t*)out, ld_out, (int)N);
}

void mfma_dense(int trans_w, const void* W, int n, int m, const void* act, i64 N_act, void* out, i64 ld_out, i64 N, void* ws, hipStream_t st) {
  const int M = trans_w ? m : n, K = trans_w ? n : m;
  const DensePlan p = pick_plan(M, N_act, K);
  DenseArgs g{};
  g.A = (const uint16_t*)W;
  g.B = (const uint16_t*)act;
  g.C = (uint16_t*)out;
  g.lda = m;
  g.ldb = N_act;
  g.ldc = ld_out;
  g.cols = (int)N;
  g.splits = p.splits;
  g.parts = (float*)ws;
  const ContractionRange range = contraction_ranges(K / BK, p.splits);
  g.ktiles = range.ktiles;
  g.longer = range.longer;
  if (p.splits > 1) {
    if (trans_w) launch_tile<false, OUT_PARTS, Tile128>(g, M, N_act, st);
    else launch_tile<true, OUT_PARTS, Tile128>(g, M, N_act, st);
    mfma_dense_reduce((const float*)ws, p.splits, M, N_act, out, ld_out, N, st);
    return;
  }
  const bool ragged = N < N_act || ld_out % 8 != 0 || ((uintptr_t)out & 15) != 0;
  if (!trans_w) {
    if (ragged) launch_dense<true, OUT_RAGGED>(g, p.tile, M, N_act, st);
    else launch_dense<true, OUT_WHOLE>(g, p.tile, M, N_act, st);
  } else {
    if (ragged) launch_dense<false, OUT_RAGGED>(g, p.tile, M, N_act, st);
    else launch_dense<false, OUT_WHOLE>(g, p.tile, M, N_act, st);
  }
}

}  // namespace poetx
