// Block gradients on the matrix cores (Sec. 3.5, mm1/mm3 backward):
//   dG_j = U'_j V'_j^T,  U'_j / V'_j = rows j*b .. j*b+b-1 of U / V gathered by the
//   side's permutation, contraction over the N tokens.
// Both operands are contracted over their contiguous (token) index.  The output
// is only nb blocks of b x b, so the token range is split over `splits`
// workgroups per tile; each writes an fp32 partial tile and a second kernel
// adds the partials in a fixed order (deterministic, no atomics).
#include "mfma_gemm.h"

namespace poetx {
namespace {

constexpr int GBM = 256, GBN = 256, GBK = 64;

struct EpiPartial {
  float* out;
  int b;
  i64 split_stride;
  __device__ void operator()(int batch, int split, int row, int col, float4 lo, float4 hi) const {   // whole 32-byte sectors
    float* p = out + split * split_stride + ((i64)batch * b + row) * b + col;
    *reinterpret_cast<float4*>(p) = lo;
    *reinterpret_cast<float4*>(p + 4) = hi;
  }
};

__global__ void reduce_partials_kernel(const float4* __restrict__ part, float4* __restrict__ out, i64 n4, int splits) {
  i64 idx = (i64)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= n4) return;
  float4 s = part[idx];
  for (int z = 1; z < splits; ++z) {
    float4 p = part[(i64)z * n4 + idx];
    s.x += p.x; s.y += p.y; s.z += p.z; s.w += p.w;
  }
  out[idx] = s;
}

int pick_splits(int d, i64 N, int b) {
  const int tiles = (d / b) * (b / GBM) * (b / GBN);
  const int ktiles = (int)(N / GBK);
  int s = 1;
  while (s * 2 * tiles <= 256 && s * 2 <= 64 && ktiles % (s * 2) == 0 && ktiles / (s * 2) >= 4) s *= 2;
  return s;
}

}  // namespace

bool mfma_blockgrad_supported(int d, i64 N, int b) {
  return (b == 256 || b == 512) && d % b == 0 && N % GBK == 0 && N >= 4 * GBK && N < (1ll << 31);
}

// The 256 x 256 tiles read every row once (b = 256) or twice and leave most CUs without one until there are many tokens; the edge kernel's 128 x 128 tiles with a split per
// 256 tokens read twice as much.  us for two sides, here / edge kernel: b = 256: 1024 features, 256 tokens 29.8 / 7.9, 4096 56.9 / 39.6; 4096 features, 2048 tokens 54 / 47,
// 8192 (2^25 elements) 107 / 88, 16384 166 / 182; 14336, 4096 155 / 153; b = 512: 1024, 256 31.0 / 8.9; 4096, 4096 84 / 76; 2048, 16384 126 / 128; 8192, 4096 (both 2^25) 130 / 139,
// 16384 372 / 424.
bool mfma_blockgrad_preferred(int d, i64 N, int b) { return mfma_blockgrad_supported(d, N, b) && (i64)d * N + (b == 512) > 1 << 25; }

size_t mfma_blockgrad_workspace_bytes(int d, i64 N, int b) {
  return (size_t)pick_splits(d, N, b) * d * b * sizeof(float);
}

void mfma_blockgrad(const void* U, i64 ldu, const void* V, i64 ldv, int d, i64 N, const int32_t* perm, int b, float* dG, void* ws, hipStream_t st) {
  const int nb = d / b;
  const int splits = pick_splits(d, N, b);
  mm::Args g{};
  g.s.A = (const uint16_t*)U;
  g.s.B = (const uint16_t*)V;
  g.s.lda = ldu;
  g.s.ldb = ldv;
  g.s.ktiles = (int)(N / GBK) / splits;
  g.tiles_m = b / GBM;
  g.tiles_n = b / GBN;
  g.perm = perm;
  g.rows_per_batch = b;
  const i64 total = (i64)nb * b * b;
  float* part = splits > 1 ? (float*)ws : dG;
  mm::launch<GBM, GBN, 2, 4, true, true, true, 4, false>(g, EpiPartial{part, b, total}, nb, splits, st);
  if (splits > 1)
    hipLaunchKernelGGL(reduce_partials_kernel, dim3(ceil_div(total / 4, 256)), dim3(256), 0, st, (const float4*)part,
                       (float4*)dG, total / 4, splits);
}

}  // namespace poetx
