// Cayley-Neumann series and its backward in fp32 for block sides up to 128, one launch each
// (Sec. 3.4, Eq. 8-9; the packed parameters in, blocks or packed gradients out).
//
// A workgroup owns 16 columns of a block, its waves 16 rows each.  Every product multiplies from the left, so column stripes never mix: a wave
// keeps its rows of the left factors in registers as matrix-core operands (v_mfma_f32_16x16x4_f32, fp32 operands and accumulation), and what moves
// from step to step are stripes of the running matrices, through LDS, one barrier per step.  The accumulator layout (lane = column, register e of row
// tile t = row 16 t + 4 (lane / 16) + e) is the B operand of the next product if the contraction index is taken in the same order: a tile
// is written as it lies in the registers and read back as four operands.
//   forward    H_1 = Q,  H_{s+1} = 2Q + Q H_s,  G = I + H_{k+1}
//   backward   with D = dL/dG, T = Q^T = -Q and c = 2, .., 2, 1 the packed gradient is the upper triangle of
//              dL/dQ - (dL/dQ)^T = sum_{s<=k} c_s sum_{i+j=s} T^i D_s T^j,   D_s = D - (-1)^s D^T
//              (the transpose of T^i D T^j is (-1)^{i+j} T^j D^T T^i): no transpose of a result, so that no stripe needs another one.
//              By Horner's rule in the left power, L = 0 .. k the right one:
//                Z_0 = D_k,  Z_L = D_k E_L + D_{k-1} F_L + T Z_{L-1},   E_L = T^L + 2 (T^{L-2} + T^{L-4} + ..),  F_L = 2 (T^{L-1} + T^{L-3} + ..)
//              and Z_k is the result.  E_L = T^L + F_{L-1} and F_L = E_{L-1} + T^{L-1} are sums of what a wave holds; their multiples of the
//              identity enter as the fp32 term of the step, 2 D_k (L even) or 2 D_{k-1} (L odd).  Four products a step.
//
// What bounds it: latency.  A step of a 64-block is 2048 cycles of matrix instructions backward (512 forward) on a quarter of the chip's
// SIMDs where a layer has 20 to 30 blocks, the rest loads and barriers.  Launches, us, a workgroup per block -> 16 columns of one: 30 blocks of 64,
// k = 4, build 8.8 -> 6.2, backward 20.5 -> 10.8 (28 blocks: 23.8 -> 11.7); whole calls, 30 blocks of 128: 39 -> 12 and 68 -> 25.
// Error of the packed gradient against 64 bits 7.3e-8 -> 4.4e-8.
#include "poetx_kernels.h"

namespace poetx {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));

__device__ inline floatx4 mfma4(float a, float b, floatx4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

struct Geometry {
  int b, side;   // stored side, live side (smaller for a ragged last block)
};

// skew(theta) into LDS, zero outside the live side.  All loads of a thread are in flight together.
template <int BP, int NTH>
__device__ __forceinline__ void load_q(float* Q, const float* theta, Geometry s, int tid) {
  constexpr int LD = BP + 4, NE = BP * BP / NTH, CH = NE < 16 ? NE : 16;
#pragma unroll
  for (int e0 = 0; e0 < NE; e0 += CH) {
    float q[CH];
#pragma unroll
    for (int e = 0; e < CH; ++e) {
      const int idx = tid + (e0 + e) * NTH, i = idx / BP, c = idx % BP;
      q[e] = i < c && c < s.side ? theta[packed_index(i, c, s.b)] : 0.f;
    }
#pragma unroll
    for (int e = 0; e < CH; ++e) {
      const int idx = tid + (e0 + e) * NTH, i = idx / BP, c = idx % BP;
      if (i <= c) Q[i * LD + c] = q[e];
      if (i < c) Q[c * LD + i] = -q[e];
    }
  }
}

// acc += A * stripe: the wave's rows of the left factor, the stripe's row tiles
template <int NT>
__device__ __forceinline__ void product(floatx4& acc, const floatx4 (&A)[NT], const floatx4* stripe, int lane) {
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const floatx4 y = stripe[t * 64 + lane];
#pragma unroll
    for (int e = 0; e < 4; ++e) acc = mfma4(A[t][e], y[e], acc);
  }
}

// Which block and stripe: stripes of a block that has fewer columns than its padded side are not launched.
struct Place {
  int lane, x, g, w;   // x: column in the stripe, row in a left operand
  int ct;
  i64 j;
};
__device__ __forceinline__ Place place(int first, int stripes) {
  Place p;
  p.lane = threadIdx.x & 63;
  p.x = p.lane & 15;
  p.g = p.lane >> 4;
  p.w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wg = first + (int)blockIdx.x;
  p.j = wg / stripes;
  p.ct = wg % stripes;
  return p;
}

template <int NT>
__global__ __launch_bounds__(64 * NT) void series_small_build_kernel(const float* __restrict__ theta, int d, int b, int k, int stripes, float* __restrict__ G,
                                                                     uint16_t* __restrict__ E, int first) {
  constexpr int BP = NT * 16, LD = BP + 4;
  extern __shared__ __attribute__((aligned(16))) float lds[];
  float* Q = lds;
  floatx4* Y = reinterpret_cast<floatx4*>(lds + BP * LD);     // two stripes of NT * 64
  const Place p = place(first, stripes);
  const Geometry s{b, block_side(d, b, (int)p.j)};
  load_q<BP, 64 * NT>(Q, theta + p.j * ((i64)b * (b - 1) / 2), s, threadIdx.x);
  __syncthreads();
  const int col = p.ct * 16 + p.x;
  floatx4 A[NT], acc, Q2;
#pragma unroll
  for (int t = 0; t < NT; ++t) A[t] = *reinterpret_cast<const floatx4*>(Q + (16 * p.w + p.x) * LD + 16 * t + 4 * p.g);
  acc = -*reinterpret_cast<const floatx4*>(Q + col * LD + 16 * p.w + 4 * p.g);   // column col of Q: minus its row
  Q2 = 2.f * acc;
  for (int step = 0; step < k; ++step) {
    floatx4* y = Y + (step & 1) * NT * 64;                    // read last before the previous barrier
    y[p.w * 64 + p.lane] = acc;
    __syncthreads();
    acc = floatx4{0.f, 0.f, 0.f, 0.f};
    product<NT>(acc, A, y, p.lane);
    acc += Q2;                                                // last: the products are small beside it, and their sum is rounded as such
  }
  const i64 bb = (i64)b * b;
  if (col >= b) return;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int i = 16 * p.w + 4 * p.g + e;
    if (i >= b) break;
    if (G) G[p.j * bb + i * b + col] = i == col ? acc[e] + 1.f : acc[e];
    if (E) {
      const uint16_t v = float_to_bf16_bits(acc[e]);
      E[p.j * 2 * bb + i * b + col] = v;
      E[p.j * 2 * bb + bb + col * b + i] = v;
    }
  }
}

struct BwdSide {
  const float* theta;
  const float* dG;       // nsplit partial block gradients, `stride` floats apart, added in order
  i64 stride;
  int nsplit, d, nb;
  float* dtheta;
};
struct BwdArgs {
  BwdSide s[2];          // blocks of the first side, then of the second
  int b, k, accumulate, stripes;
  int first;             // number of the launch's first workgroup
};

// The parts of a block's dL/dG into LDS, added in order, zero outside the live side; the loads of ZU parts are in flight together (backward calls, us,
// one part at a time / ZU: whole blocks 256 x 256, b = 32, 4096 tokens 41 / 37; stripes 512 x 512, b = 64, 8192 tokens 59 / 51).  More than two would cost whole blocks the
// registers of a fifth wave per SIMD (768 of 64, k = 4: 32.4 / 40.7 with four).
template <int BP, int NTH, int ZU>
__device__ __forceinline__ void load_d(float* D, const BwdSide& sd, i64 j, Geometry s, int tid) {
  constexpr int LD = BP + 4, NE = BP * BP / NTH;
  const float* dG = sd.dG + j * (i64)s.b * s.b;
  float v[NE];
#pragma unroll
  for (int e = 0; e < NE; ++e) v[e] = 0.f;
  int z = 0;
  auto add = [&](auto N_) {
    constexpr int N = decltype(N_)::value;
    float q[N][NE];
#pragma unroll
    for (int u = 0; u < N; ++u)
#pragma unroll
      for (int e = 0; e < NE; ++e) {
        const int idx = tid + e * NTH, i = idx / BP, c = idx % BP;
        q[u][e] = dG[(z + u) * sd.stride + (i < s.side && c < s.side ? i * s.b + c : 0)];
      }
#pragma unroll
    for (int u = 0; u < N; ++u)
#pragma unroll
      for (int e = 0; e < NE; ++e) v[e] += q[u][e];
    z += N;
  };
  while (z + ZU <= sd.nsplit) add(std::integral_constant<int, ZU>{});
  while (z < sd.nsplit) add(std::integral_constant<int, 1>{});
#pragma unroll
  for (int e = 0; e < NE; ++e) {
    const int idx = tid + e * NTH, i = idx / BP, c = idx % BP;
    D[i * LD + c] = i < s.side && c < s.side ? v[e] : 0.f;
  }
}

template <int NT>
__global__ __launch_bounds__(64 * NT) void series_small_bwd_kernel(BwdArgs a) {
  constexpr int BP = NT * 16, LD = BP + 4, NTH = 64 * NT, ST = NT * 64;
  extern __shared__ __attribute__((aligned(16))) float lds[];
  float* Q = lds;
  float* D = lds + BP * LD;
  const Place p = place(a.first, a.stripes);
  const int tid = threadIdx.x, b = a.b;
  const bool second = p.j >= a.s[0].nb;
  const BwdSide& sd = a.s[second ? 1 : 0];
  const i64 j = second ? p.j - a.s[0].nb : p.j;
  const Geometry s{b, block_side(sd.d, b, (int)j)};
  const i64 L = (i64)b * (b - 1) / 2;
  load_q<BP, NTH>(Q, sd.theta + j * L, s, tid);
  load_d<BP, NTH, NT <= 4 ? 4 : 1>(D, sd, j, s, tid);
  __syncthreads();
  const int row = 16 * p.w + p.x, col = p.ct * 16 + p.x, r0 = 16 * p.w + 4 * p.g;
  const float sk = a.k & 1 ? -1.f : 1.f;          // (-1)^k
  // left operands: T = -Q, D_k = D - (-1)^k D^T, D_{k-1} = D + (-1)^k D^T
  floatx4 AT[NT], AK[NT], AK1[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int c0 = 16 * t + 4 * p.g;
    AT[t] = -*reinterpret_cast<const floatx4*>(Q + row * LD + c0);
    const floatx4 up = *reinterpret_cast<const floatx4*>(D + row * LD + c0);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float lo = sk * D[(c0 + e) * LD + row];
      AK[t][e] = up[e] - lo;
      AK1[t][e] = up[e] + lo;
    }
  }
  // tiles of the stripe (rows r0 .. + 3 of column col): W = T^L, E, F without their multiples of the identity, Z, and the identity's terms
  floatx4 W = *reinterpret_cast<const floatx4*>(Q + col * LD + r0), E = W, F = {0.f, 0.f, 0.f, 0.f}, Z, Ck, Ck1;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float up = D[(r0 + e) * LD + col], lo = sk * D[col * LD + r0 + e];
    Z[e] = up - lo;
    Ck1[e] = 2.f * (up + lo);
  }
  Ck = 2.f * Z;
  __syncthreads();                                // Q and D are in registers: their place takes the stripes, 8 of NT KB
  floatx4* Y = reinterpret_cast<floatx4*>(lds);
  for (int step = 1; step <= a.k; ++step) {
    floatx4* y = Y + (step & 1) * 4 * ST;         // read last before the previous barrier
    const int at = p.w * 64 + p.lane;
    y[at] = E;
    y[ST + at] = F;
    y[2 * ST + at] = Z;
    y[3 * ST + at] = W;
    __syncthreads();
    Z = floatx4{0.f, 0.f, 0.f, 0.f};
    product<NT>(Z, AK, y, p.lane);
    if (step > 1) product<NT>(Z, AK1, y + ST, p.lane);       // F_1 is a multiple of the identity
    product<NT>(Z, AT, y + 2 * ST, p.lane);
    Z += step & 1 ? Ck1 : Ck;                     // last: the products are small beside it, and their sum is rounded as such
    if (step < a.k) {
      floatx4 V = {0.f, 0.f, 0.f, 0.f};
      product<NT>(V, AT, y + 3 * ST, p.lane);
      const floatx4 e = V + F;
      F = E + W;
      E = e;
      W = V;
    }
  }
  if (col >= b) return;
  float* dst = sd.dtheta + j * L;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int i = r0 + e;
    if (i >= col) break;
    const float v = col < s.side ? Z[e] : 0.f;    // dead slots of a ragged tail: zero
    float* q = dst + packed_index(i, col, b);
    *q = a.accumulate ? *q + v : v;
  }
}

// ---- whole blocks.  Many blocks fill the chip by themselves, and those of 32 are short chains anyway; then half the products count for more: a workgroup owns a block, a wave 16
// columns of it and all rows.  Backward
//   V_0 = D^T, V_m = Q V_{m-1},  W_m = 2 (V_0 + .. + V_m) - V_m,   Y_0 = D,  Y_m = W_m^T - Q Y_{m-1},  dL/dQ = Y_k,  dtheta_ic = Y_ic - Y_ci:
// half of the waves carry V and half carry Y; W_m crosses over through LDS, transposed by the read, one barrier per order (two buffers; one
// buffer and two barriers for 128, where LDS is short).
// acc = Q * Y for this wave's 16 columns.  qoff: float offset of the lane's first piece of Q; it is hidden from
// the optimiser, which would otherwise keep all of Q's fragments in registers across the orders.  128-wide
// blocks have the registers for one step's fragments only (the other waves of the SIMD hide the reads).
template <int NT>
__device__ __forceinline__ void whole_product(floatx4 (&acc)[NT], const floatx4 (&Y)[NT], const float* Q, int qoff) {
  constexpr int LD = NT * 16 + 4;
  asm volatile("" : "+v"(qoff));
  const float* qa = Q + qoff;
#pragma unroll
  for (int t = 0; t < NT; ++t) acc[t] = floatx4{0.f, 0.f, 0.f, 0.f};
  constexpr int TH = NT < 4 ? NT : 4;   // row tiles at a time
#pragma unroll
  for (int s = 0; s < NT; ++s) {
#pragma unroll
    for (int t0 = 0; t0 < NT; t0 += TH) {
      floatx4 a[TH];
#pragma unroll
      for (int t = 0; t < TH; ++t) a[t] = *reinterpret_cast<const floatx4*>(qa + (t0 + t) * 16 * LD + s * 16);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int t = 0; t < TH; ++t) acc[t0 + t] = mfma4(a[t][e], Y[s][e], acc[t0 + t]);
      if (NT == 8) __builtin_amdgcn_sched_barrier(0);
    }
  }
}

template <int NT>
__global__ __launch_bounds__(64 * NT) void series_small_build_whole_kernel(const float* __restrict__ theta, int d, int b, int k, float* __restrict__ G,
                                                                     uint16_t* __restrict__ E, int first) {
  constexpr int BP = NT * 16, LD = BP + 4;
  extern __shared__ __attribute__((aligned(16))) float lds[];
  float* Q = lds;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const i64 j = first + (int)blockIdx.x;
  const Geometry s{b, block_side(d, b, (int)j)};
  load_q<BP, 64 * NT>(Q, theta + j * ((i64)b * (b - 1) / 2), s, tid);
  __syncthreads();
  const int x = lane & 15, g = lane >> 4;
  const int col = wave * 16 + x;
  const int qoff = x * LD + 4 * g;
  floatx4 Y[NT], acc[NT], Q2[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {   // rows 16 t + 4 g + e of column col of Q: minus the row `col`
    const floatx4 r = *reinterpret_cast<const floatx4*>(Q + col * LD + 16 * t + 4 * g);
    Y[t] = -r;
    Q2[t] = -2.f * r;
  }
  for (int step = 0; step < k; ++step) {
    whole_product<NT>(acc, Y, Q, qoff);
#pragma unroll
    for (int t = 0; t < NT; ++t) Y[t] = acc[t] + Q2[t];
  }
  __syncthreads();                  // every wave is done with Q: its place takes G - I
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int e = 0; e < 4; ++e) Q[(16 * t + 4 * g + e) * LD + col] = Y[t][e];
  __syncthreads();
  const i64 bb = (i64)b * b;
#pragma unroll 8
  for (int idx = tid; idx < BP * BP; idx += 64 * NT) {
    const int i = idx / BP, c = idx % BP;
    if (i >= b || c >= b) continue;
    const float v = Q[i * LD + c];
    const int o = i * b + c;
    if (G) G[j * bb + o] = i == c ? v + 1.f : v;
    if (E) {
      E[j * 2 * bb + o] = float_to_bf16_bits(v);
      E[j * 2 * bb + bb + o] = float_to_bf16_bits(Q[c * LD + i]);
    }
  }
}

template <int NT>
__global__ __launch_bounds__(128 * NT) void series_small_bwd_whole_kernel(BwdArgs a) {
  constexpr int BP = NT * 16, LD = BP + 4, NTH = 128 * NT;
  constexpr bool TWO = NT <= 4;     // two crossing buffers
  extern __shared__ __attribute__((aligned(16))) float lds[];
  float* Q = lds;
  float* const W0 = lds + BP * LD;   // crossing buffers W0 and, where there are two, the one behind it
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wg = a.first + (int)blockIdx.x;
  const bool second = wg >= a.s[0].nb;
  const BwdSide& sd = a.s[second ? 1 : 0];
  const i64 j = second ? wg - a.s[0].nb : wg;
  const int b = a.b;
  const Geometry s{b, block_side(sd.d, b, (int)j)};
  const i64 L = (i64)b * (b - 1) / 2;
  load_q<BP, NTH>(Q, sd.theta + j * L, s, tid);
  float* D = W0;
  load_d<BP, NTH, NT <= 4 ? 2 : 1>(D, sd, j, s, tid);
  __syncthreads();
  const int x = lane & 15, g = lane >> 4;
  const bool isV = wave < NT;
  const int col = (isV ? wave : wave - NT) * 16 + x;
  const int qoff = x * LD + 4 * g;
  floatx4 Y[NT], acc[NT], S[NT];
  if (isV) {
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      Y[t] = *reinterpret_cast<const floatx4*>(D + col * LD + 16 * t + 4 * g);
      S[t] = Y[t];
    }
  } else {
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) Y[t][e] = D[(16 * t + 4 * g + e) * LD + col];
  }
  __syncthreads();                  // D's place is a crossing buffer from here on
  for (int step = 1; step <= a.k; ++step) {
    whole_product<NT>(acc, Y, Q, qoff);
    float* W = W0 + (TWO && (step & 1) ? BP * LD : 0);
    if (isV) {                      // V_m = acc; W_m goes across
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        Y[t] = acc[t];
        S[t] += acc[t];
#pragma unroll
        for (int e = 0; e < 4; ++e) W[(16 * t + 4 * g + e) * LD + col] = 2.f * S[t][e] - acc[t][e];
      }
    }
    __syncthreads();
    if (!isV) {                     // Y_m = W_m^T - Q Y_{m-1}
#pragma unroll
      for (int t = 0; t < NT; ++t) Y[t] = *reinterpret_cast<const floatx4*>(W + col * LD + 16 * t + 4 * g) - acc[t];
    }
    if (!TWO) __syncthreads();
  }
  if (TWO) __syncthreads();
  float* R = W0;
  if (!isV) {
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) R[(16 * t + 4 * g + e) * LD + col] = Y[t][e];
  }
  __syncthreads();
  float* dst = sd.dtheta + j * L;
#pragma unroll 8
  for (int idx = tid; idx < BP * BP; idx += NTH) {
    const int i = idx / BP, c = idx % BP;
    if (i < c && c < b) {
      const float v = c < s.side ? R[i * LD + c] - R[c * LD + i] : 0.f;   // dead slots of a ragged tail: zero
      float* p = dst + packed_index(i, c, b);
      *p = a.accumulate ? *p + v : v;
    }
  }
}

template <int NT>
constexpr int build_lds() { return 16 * NT * (16 * NT + 4) * 4 + 2 * NT * 1024; }
template <int NT>
constexpr int bwd_lds() {
  constexpr int in = 2 * 16 * NT * (16 * NT + 4) * 4, stripes = 8 * NT * 1024;
  return in > stripes ? in : stripes;
}
template <int NT>
constexpr int build_whole_lds() { return 16 * NT * (16 * NT + 4) * 4; }
template <int NT>
constexpr int bwd_whole_lds() { return (NT <= 4 ? 3 : 2) * 16 * NT * (16 * NT + 4) * 4; }

template <class K>
bool lds_set(K kern, int bytes) { return hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, bytes) == hipSuccess; }

// Stripes or whole blocks, by the workgroups that stripes would be.  us, whole / stripes: backward, k = 4, blocks of 64: 30 of them 12.8 / 9.5, 64: 12.8 / 9.7, 96: 12.8 / 13.4,
// 160: 13.0 / 20.5, 320: 22 / 32; of 48: 60: 12.5 / 9.4, 100: 12.5 / 13.1; of 128: 30: 66 / 25, 64: 67 / 50, 80: 67 / 70, 128: 67 / 93 (a workgroup of the stripes fills a
// CU's LDS there), at k = 1 64: 23.4 / 23.3; of 32 and less whole is the faster form of any number (16 of 32: 4.8 / 6.1; with 13 token ranges to add up 256 x 256 x 512
// backward 21.8 / 23.3).  Build, of 128: 30: 39.2 / 14.8, 64: 39.3 / 27.7, 128: 39.5 / 52.8, of 64: 30: 9.4 / 8.0, at k = 5 160: 11.0 / 10.1, 193: 10.7 / 11.4; at k = 1
// 64 of 128 17.3 / 21.5, 320 of 64 8.1 / 8.8.  Both forms of the build have the same bits; those of the backward add up in another order.
inline bool build_in_stripes(i64 nb, int b, int k) { return nb * ceil_div(b, 16) <= (b <= 64 ? (k < 3 ? 384 : 640) : k < 3 ? 256 : 512); }
inline bool bwd_in_stripes(i64 nb, int b) { return b > 32 && nb * ceil_div(b, 16) <= (b <= 64 ? 256 : 512); }

template <int NT>
void build_t(const float* theta, int d, int b, int k, float* G, uint16_t* E, hipStream_t st) {
  const i64 nb = ceil_div(d, b);
  if (!build_in_stripes(nb, b, k)) {
    static const bool configured = lds_set(series_small_build_whole_kernel<NT>, build_whole_lds<NT>());
    (void)configured;
    launch_in_rows(nb, [&](int first, unsigned count) {
      hipLaunchKernelGGL(series_small_build_whole_kernel<NT>, dim3(count), dim3(64 * NT), build_whole_lds<NT>(), st, theta, d, b, k, G, E, first);
    });
    return;
  }
  static const bool configured = lds_set(series_small_build_kernel<NT>, build_lds<NT>());
  (void)configured;
  const int stripes = ceil_div(b, 16);
  launch_in_rows(nb * stripes, [&](int first, unsigned count) {
    hipLaunchKernelGGL(series_small_build_kernel<NT>, dim3(count), dim3(64 * NT), build_lds<NT>(), st, theta, d, b, k, stripes, G, E, first);
  });
}

template <int NT>
void bwd_t(BwdArgs a, hipStream_t st) {
  const i64 nb = (i64)a.s[0].nb + a.s[1].nb;
  if constexpr (NT > 2) {
    if (bwd_in_stripes(nb, a.b)) {
      static const bool configured = lds_set(series_small_bwd_kernel<NT>, bwd_lds<NT>());
      (void)configured;
      a.stripes = ceil_div(a.b, 16);
      launch_in_rows(nb * a.stripes, [&](int first, unsigned count) {
        a.first = first;
        hipLaunchKernelGGL(series_small_bwd_kernel<NT>, dim3(count), dim3(64 * NT), bwd_lds<NT>(), st, a);
      });
      return;
    }
  }
  static const bool configured = lds_set(series_small_bwd_whole_kernel<NT>, bwd_whole_lds<NT>());
  (void)configured;
  launch_in_rows(nb, [&](int first, unsigned count) {
    a.first = first;
    hipLaunchKernelGGL(series_small_bwd_whole_kernel<NT>, dim3(count), dim3(128 * NT), bwd_whole_lds<NT>(), st, a);
  });
}

}  // namespace

// Blocks up to 128 fit: Q and one more fp32 matrix take 132 KB of LDS there.  Sides are padded to 32, 64 or 128.
bool series_small_supported(int b) { return b <= 128; }

void series_small_build(const float* theta, int d, int b, int k, float* G, void* E, hipStream_t st) {
  if (b <= 32) build_t<2>(theta, d, b, k, G, (uint16_t*)E, st);
  else if (b <= 64) build_t<4>(theta, d, b, k, G, (uint16_t*)E, st);
  else build_t<8>(theta, d, b, k, G, (uint16_t*)E, st);
}

void series_small_bwd(const SeriesSide* sides, int nsides, int b, int k, int accumulate, hipStream_t st) {
  BwdArgs a{};
  a.b = b;
  a.k = k;
  a.accumulate = accumulate;
  for (int i = 0; i < nsides; ++i)
    a.s[i] = BwdSide{sides[i].theta, sides[i].dG, sides[i].split_stride, sides[i].nsplit, sides[i].d, ceil_div(sides[i].d, b), sides[i].dtheta};
  if (b <= 32) bwd_t<2>(a, st);
  else if (b <= 64) bwd_t<4>(a, st);
  else bwd_t<8>(a, st);
}

}  // namespace poetx
