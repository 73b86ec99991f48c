// Cayley-Neumann series and its backward in fp32 for block sides up to 128, one launch each
// (Sec. 3.4, Eq. 8-9; the packed parameters in, blocks or packed gradients out).
//
// A workgroup owns one block.  Q is built from theta straight into LDS (fp32).  Every product of the chain
// multiplies by Q from the left, so column stripes of the running matrix never mix: a wave owns 16 columns
// and keeps them in registers (v_mfma_f32_16x16x4_f32, fp32 operands and accumulation).  The accumulator
// layout (lane = column, register e of row tile t = row 16 t + 4 (lane / 16) + e) is the B operand of the
// next product if the contraction index is taken in the same order, so the chain stays in the register file
// and the only LDS traffic of a product are the rows of Q, 16 bytes per four matrix instructions.
//   forward    H_1 = Q,  H_{s+1} = 2Q + Q H_s,  G = I + H_{k+1}
//   backward   V_0 = D^T, V_m = Q V_{m-1},  W_m = 2 (V_0 + .. + V_m) - V_m      (D = dL/dG)
//              Y_0 = D,   Y_m = W_m^T - Q Y_{m-1},  dL/dQ = Y_k,  dtheta_ic = Y_ic - Y_ci
// In the backward half of the waves carry V and half carry Y; W_m crosses over through LDS, transposed by
// the read, one barrier per order (two buffers; one buffer and two barriers for 128, where LDS is short).
//
// What bounds it: latency.  The plain kernels this replaces for b <= 128 spent one launch per product, 14 + 8 +
// 6 launches and 400 us for the 30 blocks of a 1376 x 512, b = 64, k = 4 layer step.
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
__device__ inline void load_q(float* Q, const float* theta, Geometry s, int tid) {
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

// acc = Q * Y for this wave's 16 columns.  qoff: float offset of the lane's first piece of Q; it is hidden from
// the optimiser, which would otherwise keep all of Q's fragments in registers across the orders.  128-wide
// blocks have the registers for one step's fragments only (the other waves of the SIMD hide the reads).
template <int NT>
__device__ inline void product(floatx4 (&acc)[NT], const floatx4 (&Y)[NT], const float* Q, int qoff) {
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
__global__ __launch_bounds__(64 * NT) void series_small_build_kernel(const float* __restrict__ theta, int d, int b, int k, float* __restrict__ G,
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
    product<NT>(acc, Y, Q, qoff);
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

struct BwdSide {
  const float* theta;
  const float* dG;       // nsplit partial block gradients, `stride` floats apart, added in order
  i64 stride;
  int nsplit, d, nb;
  float* dtheta;
};
struct BwdArgs {
  BwdSide s[2];          // blocks of the first side, then of the second
  int b, k, accumulate;
  int first;             // block of the launch's first workgroup
};

template <int NT>
__global__ __launch_bounds__(128 * NT) void series_small_bwd_kernel(BwdArgs a) {
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
  const float* dG = sd.dG + j * (i64)b * b;
  {   // the parts of D, added in order; the loads of a thread's elements are in flight together
    constexpr int NE = BP * BP / NTH;
    float v[NE];
#pragma unroll
    for (int e = 0; e < NE; ++e) v[e] = 0.f;
    for (int z = 0; z < sd.nsplit; ++z) {
      const float* part = dG + z * sd.stride;
#pragma unroll
      for (int e = 0; e < NE; ++e) {
        const int idx = tid + e * NTH, i = idx / BP, c = idx % BP;
        if (i < b && c < b) v[e] += part[i * b + c];
      }
    }
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      const int idx = tid + e * NTH;
      D[(idx / BP) * LD + idx % BP] = v[e];
    }
  }
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
    product<NT>(acc, Y, Q, qoff);
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
constexpr int build_lds() { return 16 * NT * (16 * NT + 4) * 4; }
template <int NT>
constexpr int bwd_lds() { return (NT <= 4 ? 3 : 2) * 16 * NT * (16 * NT + 4) * 4; }

template <int NT>
void build_t(const float* theta, int d, int b, int k, float* G, uint16_t* E, hipStream_t st) {
  static const bool configured = hipFuncSetAttribute((const void*)series_small_build_kernel<NT>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                                     build_lds<NT>()) == hipSuccess;
  (void)configured;
  launch_in_rows(ceil_div(d, b), [&](int first, unsigned count) {
    hipLaunchKernelGGL(series_small_build_kernel<NT>, dim3(count), dim3(64 * NT), build_lds<NT>(), st, theta, d, b, k, G, E, first);
  });
}

template <int NT>
void bwd_t(BwdArgs a, hipStream_t st) {
  static const bool configured = hipFuncSetAttribute((const void*)series_small_bwd_kernel<NT>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                                     bwd_lds<NT>()) == hipSuccess;
  (void)configured;
  launch_in_rows((i64)a.s[0].nb + a.s[1].nb, [&](int first, unsigned count) {
    a.first = first;
    hipLaunchKernelGGL(series_small_bwd_kernel<NT>, dim3(count), dim3(128 * NT), bwd_lds<NT>(), st, a);
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
