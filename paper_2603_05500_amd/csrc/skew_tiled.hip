// Q = skew(theta) and its adjoint on the packed parameters (Sec. 3.4), tile by tile.
//   materialise: Q[i][c] = +theta[idx(i, c)] for i < c, -theta[idx(c, i)] for i > c, 0 on the diagonal
//   project:     dtheta[idx(i, c)] (+)= M[i][c] - M[c][i] for i < c
// idx is the row-major strict upper triangle, so a row segment of the upper triangle is contiguous in
// theta while its mirror image is a column.  A workgroup takes a 64 x 64 tile (I, J), I <= J, together
// with its mirror tile (J, I) and passes the transposed half through LDS: every global access of both
// kernels runs along contiguous addresses.  For blocks whose side is a multiple of 64 and dimensions
// that are whole blocks (the matrix-core paths); other shapes keep the element-wise kernels.
#include "poetx_kernels.h"

namespace poetx {
namespace {

constexpr int ST = 64;

// tile pair p of the upper triangle (diagonal included) of a T x T tile grid, row by row
__device__ inline void pair_decode(int p, int T, int& I, int& J) {
  I = 0;
  while (p >= T - I) {
    p -= T - I;
    ++I;
  }
  J = I + p;
}

// The upper triangle's tile (I, J) of a block into LDS, zeros on and below the diagonal.  All 16 loads of a thread are in
// flight together (four at a time, a launch over 32 blocks of 256 took 10.8 us instead of 6.9).
__device__ __forceinline__ void load_tile(float (&tile)[ST][ST + 1], const float* th, int I, int J, int b) {
  const int c = threadIdx.x & 63, r0 = threadIdx.x >> 6;
  float v[ST / 4];
#pragma unroll
  for (int s = 0; s < ST / 4; ++s) {
    const int i = I * ST + r0 + 4 * s, col = J * ST + c;
    v[s] = i < col ? th[packed_index(i, col, b)] : 0.f;
  }
#pragma unroll
  for (int s = 0; s < ST / 4; ++s) tile[r0 + 4 * s][c] = v[s];
  __syncthreads();
}

__global__ __launch_bounds__(256) void skew_materialize_tiled_kernel(const float* __restrict__ theta, int b, float* __restrict__ Qf,
                                                                     uint16_t* __restrict__ Qb, uint16_t* __restrict__ Tb) {
  __shared__ float tile[ST][ST + 1];
  int I, J;
  pair_decode(blockIdx.x, b / ST, I, J);
  const i64 j = blockIdx.y;
  load_tile(tile, theta + j * ((i64)b * (b - 1) / 2), I, J, b);
  const int c = threadIdx.x & 63, r0 = threadIdx.x >> 6;
  auto put = [&](i64 at, float q) {
    if (Qf) Qf[at] = q;
    if (Qb) Qb[at] = float_to_bf16_bits(q);
    if (Tb) Tb[at] = float_to_bf16_bits(-q);
  };
#pragma unroll 4
  for (int r = r0; r < ST; r += 4) {
    float q = tile[r][c];                               // strictly above the diagonal where I < J
    if (I == J) q = c > r ? tile[r][c] : (c < r ? -tile[c][r] : 0.f);
    put((j * b + I * ST + r) * b + J * ST + c, q);
    if (I != J) put((j * b + J * ST + r) * b + I * ST + c, -tile[c][r]);   // Q[J*64 + r][I*64 + c] = -Q[I*64 + c][J*64 + r]
  }
}

// What the on-chip chains of b = 256 read, as matrix-core fragments [block][row tile][k step][lane][8], lane 32h + r holding of row r
// of the tile the contraction elements 16s + 4h + {0, 1, 2, 3, 8, 9, 10, 11}: bf16(Q), or for the backward bf16(-Q) and bf16(D) (D given).
// Blocks 0 .. nb0 - 1 come from theta and D, the rest from theta2 and D2.
__global__ __launch_bounds__(256) void skew_materialize_chain_kernel(const float* __restrict__ theta, const float* __restrict__ theta2, int nb0,
                                                                     uint16_t* __restrict__ Qf, const float* __restrict__ D,
                                                                     const float* __restrict__ D2, uint16_t* __restrict__ Df) {
  constexpr int B = 256, PAIRS = (B / ST) * (B / ST + 1) / 2;
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  typedef float f32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));
  __shared__ float tile[ST][ST + 1];
  const i64 j = blockIdx.y;
  const int tid = threadIdx.x;
  if (blockIdx.x >= PAIRS) {                            // a row tile of D
    const int w = blockIdx.x - PAIRS;
    const float* d = (j < nb0 ? D + j * B * B : D2 + (j - nb0) * B * B) + (32 * w + (tid & 31)) * B + 16 * (tid >> 6) + 4 * ((tid >> 5) & 1);
    f32x4_a4 lo[4], hi[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      lo[i] = *reinterpret_cast<const f32x4_a4*>(d + 64 * i);
      hi[i] = *reinterpret_cast<const f32x4_a4*>(d + 64 * i + 8);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      u32x4 o;
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        o[e] = float_to_bf16_bits(lo[i][2 * e]) | (uint32_t)float_to_bf16_bits(lo[i][2 * e + 1]) << 16;
        o[2 + e] = float_to_bf16_bits(hi[i][2 * e]) | (uint32_t)float_to_bf16_bits(hi[i][2 * e + 1]) << 16;
      }
      *reinterpret_cast<u32x4*>(Df + (((j * 8 + w) * 16 + 4 * i + (tid >> 6)) * 64 + (tid & 63)) * 8) = o;
    }
    return;
  }
  int I, J;
  pair_decode(blockIdx.x, B / ST, I, J);
  load_tile(tile, (j < nb0 ? theta + j * (B * (B - 1) / 2) : theta2 + (j - nb0) * (B * (B - 1) / 2)), I, J, B);
  const float sign = D ? -1.f : 1.f;
#pragma unroll 1
  for (int m = 0; m < (I == J ? 1 : 2); ++m) {          // the tile, then its mirror image
    auto q = [&](int r, int c) {
      if (m) return -sign * tile[c][r];
      return I != J || c > r ? sign * tile[r][c] : (c < r ? -sign * tile[c][r] : 0.f);
    };
    const int R = m ? J : I, C = m ? I : J;
#pragma unroll
    for (int p = 0; p < 2; ++p) {                       // row tile 2R + p, k steps 4C + s
      const int s = tid >> 6, r = 32 * p + (tid & 31), c = 16 * s + 4 * ((tid >> 5) & 1);
      u32x4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int cc = c + 8 * (e >> 1) + 2 * (e & 1);
        o[e] = float_to_bf16_bits(q(r, cc)) | (uint32_t)float_to_bf16_bits(q(r, cc + 1)) << 16;
      }
      *reinterpret_cast<u32x4*>(Qf + (((j * 8 + 2 * R + p) * 16 + 4 * C + s) * 64 + (tid & 63)) * 8) = o;
    }
  }
}

// M of the on-chip chains (b = 256, 32 x 32 tiles [block][row tile][column tile][1024]: element (r, c) of a tile at
// 256 (r / 8) + 128 ((r / 4) & 1) + 4 c + (r & 3)) -> packed gradients; blocks 0 .. nb0 - 1 go to dtheta, the rest to dtheta2
__global__ __launch_bounds__(256) void skew_project_chain_kernel(const float* __restrict__ M, int nb0, float* __restrict__ dtheta,
                                                                 float* __restrict__ dtheta2, int accumulate) {
  constexpr int B = 256;
  __shared__ float up[ST][ST + 1], lo[ST][ST + 1];
  int I, J;
  pair_decode(blockIdx.x, B / ST, I, J);
  const i64 j = blockIdx.y;
  const int tid = threadIdx.x;
  {
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    const int c = tid & 31, r = 8 * (tid >> 6) + 4 * ((tid >> 5) & 1);
    f32x4 u[4], l[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      u[q] = *reinterpret_cast<const f32x4*>(M + ((j * 8 + 2 * I + (q >> 1)) * 8 + 2 * J + (q & 1)) * 1024 + tid * 4);
      l[q] = *reinterpret_cast<const f32x4*>(M + ((j * 8 + 2 * J + (q >> 1)) * 8 + 2 * I + (q & 1)) * 1024 + tid * 4);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        up[32 * (q >> 1) + r + e][32 * (q & 1) + c] = u[q][e];
        lo[32 * (q >> 1) + r + e][32 * (q & 1) + c] = l[q][e];
      }
  }
  __syncthreads();
  float* dt = (j < nb0 ? dtheta + j * (B * (B - 1) / 2) : dtheta2 + (j - nb0) * (B * (B - 1) / 2));
  const int c = tid & 63, r0 = tid >> 6;
#pragma unroll 4
  for (int r = r0; r < ST; r += 4) {
    const int i = I * ST + r, col = J * ST + c;
    if (i < col) {
      const float v = up[r][c] - lo[c][r];   // M[i][col] - M[col][i]
      float* dst = dt + packed_index(i, col, B);
      *dst = accumulate ? *dst + v : v;
    }
  }
}

// blocks 0 .. nb0 - 1 of M go to dtheta, the rest to dtheta2
__global__ __launch_bounds__(256) void skew_project_tiled_kernel(const float* __restrict__ M, int b, int nb0, float* __restrict__ dtheta,
                                                                 float* __restrict__ dtheta2, int accumulate) {
  __shared__ float up[ST][ST + 1], lo[ST][ST + 1];
  int I, J;
  pair_decode(blockIdx.x, b / ST, I, J);
  const i64 j = blockIdx.y;
  const float* Mj = M + j * (i64)b * b;
  float* dt = (j < nb0 ? dtheta + j * ((i64)b * (b - 1) / 2) : dtheta2 + (j - nb0) * ((i64)b * (b - 1) / 2));
  const int c = threadIdx.x & 63, r0 = threadIdx.x >> 6;
#pragma unroll 16
  for (int r = r0; r < ST; r += 4) {
    up[r][c] = Mj[(i64)(I * ST + r) * b + J * ST + c];
    lo[r][c] = Mj[(i64)(J * ST + r) * b + I * ST + c];
  }
  __syncthreads();
#pragma unroll 4
  for (int r = r0; r < ST; r += 4) {
    const int i = I * ST + r, col = J * ST + c;
    if (i < col) {
      const float v = up[r][c] - lo[c][r];   // M[i][col] - M[col][i]
      float* dst = dt + packed_index(i, col, b);
      *dst = accumulate ? *dst + v : v;
    }
  }
}

}  // namespace

bool skew_tiled_supported(int b, i64 d) { return b % ST == 0 && d % b == 0; }

void skew_materialize_tiled_launch(const float* theta, int b, i64 nb, float* Qf, uint16_t* Qb, uint16_t* Tb, hipStream_t st) {
  const int T = b / ST;
  hipLaunchKernelGGL(skew_materialize_tiled_kernel, dim3(T * (T + 1) / 2, (unsigned)nb), dim3(256), 0, st, theta, b, Qf, Qb, Tb);
}

void skew_materialize_chain_launch(const float* theta0, i64 nb0, const float* theta1, i64 nb1, uint16_t* Qf, const float* D0, const float* D1, uint16_t* Df,
                                   hipStream_t st) {
  constexpr int T = 256 / ST;
  hipLaunchKernelGGL(skew_materialize_chain_kernel, dim3(T * (T + 1) / 2 + (D0 ? 8 : 0), (unsigned)(nb0 + nb1)), dim3(256), 0, st, theta0, theta1, (int)nb0, Qf, D0, D1, Df);
}

void skew_project_chain_launch(const float* M, i64 nb0, float* dtheta0, i64 nb1, float* dtheta1, int accumulate, hipStream_t st) {
  constexpr int T = 256 / ST;
  hipLaunchKernelGGL(skew_project_chain_kernel, dim3(T * (T + 1) / 2, (unsigned)(nb0 + nb1)), dim3(256), 0, st, M, (int)nb0, dtheta0, dtheta1, accumulate);
}

void skew_project_tiled_launch(const float* M, int b, i64 nb, float* dtheta, int accumulate, hipStream_t st) {
  const int T = b / ST;
  hipLaunchKernelGGL(skew_project_tiled_kernel, dim3(T * (T + 1) / 2, (unsigned)nb), dim3(256), 0, st, M, b, (int)nb, dtheta, (float*)nullptr, accumulate);
}

void skew_project_sides_launch(const float* M, int b, i64 nb0, float* dtheta0, i64 nb1, float* dtheta1, int accumulate, hipStream_t st) {
  const int T = b / ST;
  hipLaunchKernelGGL(skew_project_tiled_kernel, dim3(T * (T + 1) / 2, (unsigned)(nb0 + nb1)), dim3(256), 0, st, M, b, (int)nb0, dtheta0, dtheta1, accumulate);
}

}  // namespace poetx
