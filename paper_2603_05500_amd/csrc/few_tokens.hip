// The forward of a handful of tokens (generation): bf16, up to 32 of them, whole blocks of 64, 128, 256 or 512.
//     A = R^T X        apply_few_kernel, A kept token major
//     B = W A          dense_few_kernel
//     Z = P^T B        apply_few_kernel
// X and Z are read and written in the caller's layout, element by element where that is token major.
//
// What bounds it: latency.  A launch is some 3 us, the weight of 2048 x 2048 is read in 2; so each kernel is one chain of load,
// LDS, matrix product, store with all of a wave's loads in flight at once, and nothing is split over workgroups that would
// need another launch to add it up: the waves of a workgroup split the contraction and meet in LDS.  2048 x 2048, b = 256, 16 token-major tokens,
// us: the edge product's tiles in two stages, with its split contraction and reduction 12.3 + 4.9 + 4.7 + 8.0 -> 4.9 + 6.1 + 4.1.
#include "edge_gemm.h"

namespace poetx {
namespace {

using mm::bf16x8;
typedef float floatx4 __attribute__((ext_vector_type(4)));
using edge::u32x4;

// eight elements, aligned as elements only: one load all the same
__device__ __forceinline__ bf16x8 load8(const uint16_t* p) { return __builtin_bit_cast(bf16x8, edge::load16(p)); }

// 64 rows of a block per workgroup, 16 per wave, NT * 16 tokens.  The wave's rows of op(E) are its fragments; the block's gathered features
// lie in LDS token by token.  out = V + E V: the identity part is added in fp32 from there.
template <int B, int NT, bool V_TM, bool OUT_TM>
__global__ __launch_bounds__(256) void apply_few_kernel(const uint16_t* __restrict__ V, i64 ldv, uint16_t* __restrict__ out, i64 ldo, int N,
                                                        const int32_t* __restrict__ perm, const uint16_t* __restrict__ blocks, int trans) {
  constexpr int KS = B / 32, LD = B + 8, NF = (B + 255) / 256;
  __shared__ __attribute__((aligned(16))) uint16_t xs[NT * 16 * LD];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j = blockIdx.x / (B / 64), r0 = (blockIdx.x % (B / 64)) * 64 + wave * 16;
  const int x = lane & 15, g = lane >> 4;
  const int32_t* pm = perm + (i64)j * B;
  i64 pf[NF];
#pragma unroll
  for (int i = 0; i < NF; ++i) pf[i] = tid + 256 * i < B ? pm[tid + 256 * i] : 0;
  const uint16_t* Eb = blocks + ((i64)j * 2 + (trans ? 1 : 0)) * B * B + (r0 + x) * B + 8 * g;
  bf16x8 fa[KS];
#pragma unroll
  for (int s = 0; s < KS; ++s) fa[s] = load8(Eb + 32 * s);
  i64 at[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) at[e] = pm[r0 + 4 * g + e];
#pragma unroll
  for (int i = 0; i < NF; ++i) {
    const int f = tid + 256 * i;
    if (f >= B) break;
    if constexpr (V_TM) {
      uint16_t v[NT * 16];
#pragma unroll
      for (int t = 0; t < NT * 16; ++t) v[t] = t < N ? V[t * ldv + pf[i]] : 0;
#pragma unroll
      for (int t = 0; t < NT * 16; ++t) xs[t * LD + f] = v[t];
    } else {
      u32x4 v[NT * 2];
#pragma unroll
      for (int c = 0; c < NT * 2; ++c)
        v[c] = N < 8 ? edge::load_branched(V + pf[i] * ldv, 8 * c, N, true) : edge::mask_raw(edge::load_raw(V + pf[i] * ldv, 8 * c, N), 8 * c, N, true);
#pragma unroll
      for (int t = 0; t < NT * 16; ++t) xs[t * LD + f] = (uint16_t)(v[t >> 3][(t >> 1) & 3] >> (16 * (t & 1)));
    }
  }
  __syncthreads();
  floatx4 acc[NT];
#pragma unroll
  for (int c = 0; c < NT; ++c) acc[c] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < KS; ++s)
#pragma unroll
    for (int c = 0; c < NT; ++c)
      acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[s], *reinterpret_cast<const bf16x8*>(xs + (16 * c + x) * LD + 32 * s + 8 * g), acc[c], 0, 0, 0);
  // lane (token x, g), register e: row 4g + e
#pragma unroll
  for (int c = 0; c < NT; ++c) {
    const int t = 16 * c + x;
    if (t >= N) continue;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float y = acc[c][e] + bf16_bits_to_float(xs[t * LD + r0 + 4 * g + e]);
      out[OUT_TM ? t * ldo + at[e] : at[e] * ldo + t] = (uint16_t)mm::pack2_bf16(y, 0.f);
    }
  }
}

// out (M x cols, columns from N on zero) = W (M x K) act^T, act token major: RT * 16 rows per workgroup, the contraction in NW ranges of whole
// k steps of 32.
template <int RT, int NT, int NW>
__global__ __launch_bounds__(64 * NW) void dense_few_kernel(const uint16_t* __restrict__ W, int K, const uint16_t* __restrict__ act,
                                                            uint16_t* __restrict__ out, i64 ldo, int N, int cols) {
  __shared__ float part[NW][RT * NT * 256];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int x = lane & 15, g = lane >> 4;
  const int S = K / 32, s0 = S * wave / NW, s1 = S * (wave + 1) / NW;
  const uint16_t* w = W + ((i64)blockIdx.x * (RT * 16) + x) * K + 8 * g;
  const uint16_t* a[NT];
#pragma unroll
  for (int c = 0; c < NT; ++c) a[c] = act + (i64)(16 * c + x < N ? 16 * c + x : N - 1) * K + 8 * g;   // columns past N go nowhere
  floatx4 acc[RT][NT];
#pragma unroll
  for (int r = 0; r < RT; ++r)
#pragma unroll
    for (int c = 0; c < NT; ++c) acc[r][c] = floatx4{0.f, 0.f, 0.f, 0.f};
  auto steps = [&](int s, auto U_) {        // that many k steps, their loads in flight together
    constexpr int U = decltype(U_)::value;
    bf16x8 fw[U][RT], fb[U][NT];
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int r = 0; r < RT; ++r) fw[u][r] = load8(w + (i64)r * 16 * K + 32 * (s + u));
#pragma unroll
      for (int c = 0; c < NT; ++c) fb[u][c] = load8(a[c] + 32 * (s + u));
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int c = 0; c < NT; ++c) acc[r][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[u][r], fb[u][c], acc[r][c], 0, 0, 0);
  };
  int s = s0;
  for (; s + 8 <= s1; s += 8) steps(s, std::integral_constant<int, 8>{});
  for (; s < s1; ++s) steps(s, std::integral_constant<int, 1>{});
#pragma unroll
  for (int r = 0; r < RT; ++r)
#pragma unroll
    for (int c = 0; c < NT; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e) part[wave][(r * 16 + 4 * g + e) * (16 * NT) + 16 * c + x] = acc[r][c][e];
  __syncthreads();
  for (int i = tid; i < RT * NT * 256; i += 64 * NW) {
    const int r = i / (16 * NT), t = i % (16 * NT);
    float y = 0.f;
#pragma unroll
    for (int z = 0; z < NW; ++z) y += part[z][i];
    if (t < cols) out[((i64)blockIdx.x * (RT * 16) + r) * ldo + t] = t < N ? (uint16_t)mm::pack2_bf16(y, 0.f) : 0;
  }
}

template <int NT, bool V_TM, bool OUT_TM>
void launch_apply(const uint16_t* V, i64 ldv, uint16_t* out, i64 ldo, int d, int N, const int32_t* perm, const uint16_t* E, int b, int trans, hipStream_t st) {
  auto kern = b == 64 ? apply_few_kernel<64, NT, V_TM, OUT_TM> : b == 128 ? apply_few_kernel<128, NT, V_TM, OUT_TM>
            : b == 256 ? apply_few_kernel<256, NT, V_TM, OUT_TM> : apply_few_kernel<512, NT, V_TM, OUT_TM>;
  hipLaunchKernelGGL(kern, dim3((unsigned)(d / 64)), dim3(256), 0, st, V, ldv, out, ldo, N, perm, E, trans);
}

}  // namespace

// Every workgroup reads all of A, its waves an eighth of the contraction each, one group of loads after the other: what loses is tokens times the
// contraction, where the edge kernels split; the second sixteen tokens double it.  Whole forwards, us, the edge kernels / these, feature major, token major (large weights
// from memory): 2048 x 2048, b = 256, one token 20.3 / 11.1, 20.4 / 11.0, 16: 20.5 / 13.3, 28.7 / 14.6, 32: 19.0 / 16.8, 29.0 / 19.2; b = 128, 16: 18.9 / 11.8,
// 25.5 / 13.0; b = 64: 18.2 / 11.4, 24.2 / 12.5; 4096 x 4096, b = 512, 16: 29.1 / 22.7, 41.6 / 26.1, 32: 27.0 / 30.3, 40.7 / 38.2; 14336 x 4096, 16: 44.3 / 40.8,
// 56.9 / 41.8; 4096 x 14336, 4: 46.7 / 34.4, 49.6 / 34.6, 8: 42.8 / 37.6, 52.3 / 38.4; 512 x 3328, 25 token-major tokens
// 28.0 / 19.8.  Refused: 512 x 14336, 16: 22.6 / 33.7, 32: 26.2 / 48 (feature major); 2048 x 8192, 32: 27.9 / 36.6; 10240 x 8192, 16: 50.5 / 58.7; 4096 x 14336, 16: 42.9 / 44.2.
bool few_tokens_supported(int n, int m, int b, i64 N) {
  return (b == 64 || b == 128 || b == 256 || b == 512) && n % b == 0 && m % b == 0 && n < (1 << 22) && m < (1 << 22) &&
         (N <= 16 || (N <= 32 && (i64)n * m <= 1 << 24)) && m * N <= (n < 1024 ? 3 << 15 : n > 8192 ? 1 << 16 : 1 << 17);
}

void few_apply(const void* V, i64 ldv, bool v_tm, void* out, i64 ldo, bool out_tm, int d, int N, const int32_t* perm, const void* E, int b, int trans,
               hipStream_t st) {
  auto f = N <= 16 ? (v_tm ? launch_apply<1, true, true> : out_tm ? launch_apply<1, false, true> : launch_apply<1, false, false>)
                   : (v_tm ? launch_apply<2, true, true> : out_tm ? launch_apply<2, false, true> : launch_apply<2, false, false>);
  f((const uint16_t*)V, ldv, (uint16_t*)out, ldo, d, N, perm, (const uint16_t*)E, b, trans, st);
}

void few_dense(const void* W, int M, int K, const void* act, void* out, i64 ldo, int N, int cols, hipStream_t st) {
  auto go = [&](auto kern, int rt, int nw) {
    hipLaunchKernelGGL(kern, dim3((unsigned)(M / (16 * rt))), dim3(64 * nw), 0, st, (const uint16_t*)W, K, (const uint16_t*)act, (uint16_t*)out, ldo, N, cols);
  };
  // Every workgroup reads all of act (from L2): four row tiles each where that leaves enough workgroups.  Forwards of M x 4096, one tile / four, us: 14336, 8 tokens
  // 41.0 / 37.8, 16: 45.3 / 39.2; 10240, 8: 32.1 / 35.2, 16: 37.6 / 37.1; 8192 x 8192, 16: 47.7 / 56.5.
  const bool tall = M >= 12288 && N > 6;
  if (N <= 16) tall ? go(dense_few_kernel<4, 1, 8>, 4, 8) : go(dense_few_kernel<1, 1, 8>, 1, 8);
  else go(dense_few_kernel<1, 2, 8>, 1, 8);
}

}  // namespace poetx
