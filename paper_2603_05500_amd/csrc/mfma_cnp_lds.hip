// Cayley-Neumann series and its backward for b = 256 on chip (Sec. 3.4, Eq. 8-9): one launch runs the whole chain of a
// block's column stripe.
//
// Every quantity of the series is a matrix that is multiplied from the left, step by step, and whose column stripes do not mix:
//   forward    H_1 = Q,    H_{s+1} = 2Q + Q H_s,       G = I + H_{k+1}
//   backward   U_1 = T,    U_{m+1} = T + T U_m,        Z_0 = D,  Z_m = D + D U_m + T Z_{m-1},   dL/dQ = Z_k + Z_{k-1}
// with D = dL/dG and T = Q^T = -Q.  (U_m = T + .. + T^m, so Z_m = sum_{i+j<=m} T^i D T^j, and with c = 2, .., 2, 1 dL/dQ = sum_p c_p
// sum_{i+j=p-1} T^i D T^j = Z_k + Z_{k-1}.  Carrying D T^j as D U_m takes a third product per step, but keeps the right factors on
// the left of a stripe as well: with P_m = D + P_{m-1} T instead, P_m is made of row stripes, and every one of the k of them had to go through
// memory in fp32, 420 MB each way for 320 blocks.)
//
// A workgroup owns 32 columns of a block, its eight waves 32 rows each.  A wave keeps its rows of the left factors (bf16 Q, or T and D) in
// registers as matrix-core fragments for the whole chain (64 registers each); what moves from step to step are the 256 x 32 stripes of the
// running matrices, 16 KB of bf16 each through LDS, two buffers and one barrier per step.  The products take the contraction index permuted inside
// groups of 16 (k = 16s + 8a + 4h + j at fragment slot 8h + 4a + j): registers 8u .. 8u + 7 of an accumulator tile then ARE a
// fragment of the next product, so a stripe is written as whole fragments and read back as they lie.  The fp32 term of a step is the C
// operand of its first matrix instruction and costs nothing.
//
// What bounds it: up to 32 blocks (256 workgroups, one per CU) latency: some 6 us of launch, fragments and first terms, then 0.9 us a step
// forward, 2.2 backward, of which 1024 and 3072 cycles are matrix instructions; for many blocks forward the traffic of E, backward the steps
// themselves (one workgroup per CU: two factors in registers).  us at k = 5, with all of Q in LDS, 128 columns of a chain in the registers of
// four waves, and P_m through memory -> so: forward launch 32 blocks 22 -> 9.9, 320: 84 -> 60; backward launches 32: 28 + 30 -> 18, 320:
// 115 + 117 -> 160; whole calls, build 32: 31 -> 16, 320: 111 -> 75, backward 32: 65 -> 31, 320: 283 -> 216.  The forward takes its 2Q
// from theta itself: materialised in fp32 it cost 16 us of 320 blocks' 36.  Several stripes per workgroup, one after the other, save the
// fragments' loads but not time (320 blocks: 237 us one, 240 two, 251 four).
//
// Precision as in the tiled kernels: products in bf16 with fp32 accumulation, the dominant
// terms (2Q, D, T) enter in fp32.
#include "mfma_gemm.h"

namespace poetx {
namespace {

using mm::bf16x8;
using mm::floatx16;
using mm::lds_barrier;

constexpr int LB = 256;                  // block side
constexpr int NT = LB / 32;              // row tiles = waves = column stripes
constexpr int NKS = LB / 16;             // k steps of a product
constexpr int Y_LDS = LB * 32 * 2;       // a stripe of a running matrix

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ bf16x8 negate(bf16x8 v) {
  u32x4 u = __builtin_bit_cast(u32x4, v);
  u ^= 0x80008000u;
  return __builtin_bit_cast(bf16x8, u);
}

__device__ __forceinline__ bf16x8 pack8(const floatx16& a, int u) {
  u32x4 r;
#pragma unroll
  for (int e = 0; e < 4; ++e) r[e] = mm::pack2_bf16(a[8 * u + 2 * e], a[8 * u + 2 * e + 1]);
  return __builtin_bit_cast(bf16x8, r);
}

// Where a wave of a chain stands.  The eight stripes of a block have ids 8 apart: one XCD, whose L2 brings the block's fragments in once.
struct Place {
  int lane, n, h;      // n, h: column inside the stripe and row half of the accumulator layout
  int w, ct;           // row tile, column stripe
  int j;               // block
};
__device__ __forceinline__ Place place() {
  const int tid = threadIdx.x, id = blockIdx.x;
  Place p;
  p.lane = tid & 63;
  p.n = p.lane & 31;
  p.h = p.lane >> 5;
  p.w = __builtin_amdgcn_readfirstlane(tid >> 6);
  p.ct = (id >> 3) & 7;
  p.j = (id >> 6) * 8 + (id & 7);
  return p;
}

// Tile (w, ct) of f * Q in accumulator layout (lane (n, h), register 4g + e: element (i, c) = (32w + 8g + 4h + e, 32ct + n)) from the block's
// packed triangle
__device__ __forceinline__ void q_tile(floatx16& v, const float* th, const Place& p, float f) {
  const int c = 32 * p.ct + p.n, i0 = 32 * p.w + 4 * p.h;
  if (p.w > p.ct) {          // below the diagonal: minus the mirror image, whose packed row runs along i
    const float* row = th + (c * LB - c * (c + 1) / 2 - c - 1) + i0;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const f32x4_a4 x = *reinterpret_cast<const f32x4_a4*>(row + 8 * g);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[4 * g + e] = -f * x[e];
    }
  } else {
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int i = i0 + 8 * (q >> 2) + (q & 3), lo = i < c ? i : c, hi = i < c ? c : i;
      const float t = th[lo < hi ? lo * LB - lo * (lo + 1) / 2 + hi - lo - 1 : 0];   // an address on the diagonal too: no branch around a load
      v[q] = i < c ? f * t : i > c ? -f * t : 0.f;
    }
  }
}

__device__ __forceinline__ bf16x8 fragment(const char* y, int s, int lane) { return *reinterpret_cast<const bf16x8*>(y + s * 1024 + lane * 16); }
__device__ __forceinline__ void put(char* y, const floatx16& v, const Place& p) {
#pragma unroll
  for (int u = 0; u < 2; ++u) *reinterpret_cast<bf16x8*>(y + (2 * p.w + u) * 1024 + p.lane * 16) = pack8(v, u);
}

// ---- forward
struct BuildArgs {
  const uint16_t* Qf;      // bf16(Q) of all blocks as fragments: [block][row tile][k step][lane][8]
  const float* theta;
  int k, nb;
  float* G;                // I + H, [nb][LB][LB] (nullable)
  uint16_t* E;             // bf16 pair [nb][2][LB][LB] (nullable)
};

__global__ __launch_bounds__(512, 4) void cnp_build_kernel(BuildArgs a) {
  __shared__ __attribute__((aligned(16))) char lds[2 * Y_LDS];
  const Place p = place();
  if (p.j >= a.nb) return;
  const int lane = p.lane, n = p.n, h = p.h, w = p.w, ct = p.ct;
  const i64 blk = (i64)p.j * LB * LB;
  const bf16x8* qf = reinterpret_cast<const bf16x8*>(a.Qf + blk) + lane;
  bf16x8 A[NKS];
#pragma unroll
  for (int s = 0; s < NKS; ++s) A[s] = qf[(w * NKS + s) * 64];
  floatx16 acc, C;
  q_tile(C, a.theta + (i64)p.j * (LB * (LB - 1) / 2), p, 2.f);
  // column n of Q as row n of the stripe's own tile (Q[k][c] = -Q[c][k]): same slots
#pragma unroll
  for (int u = 0; u < 2; ++u)
    *reinterpret_cast<bf16x8*>(lds + (2 * w + u) * 1024 + lane * 16) = negate(qf[(ct * NKS + 2 * w + u) * 64]);
  lds_barrier();
  for (int step = 1; step <= a.k; ++step) {
    const char* y = lds + ((step - 1) & 1) * Y_LDS;
    constexpr int DEPTH = 4;     // fragments of the stripe in flight
    bf16x8 f[DEPTH];
#pragma unroll
    for (int s = 0; s < DEPTH; ++s) f[s] = fragment(y, s, lane);
#pragma unroll
    for (int s = 0; s < NKS; ++s) {
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[s], f[s % DEPTH], s == 0 ? C : acc, 0, 0, 0);
      if (s + DEPTH < NKS) f[s % DEPTH] = fragment(y, s + DEPTH, lane);
      __builtin_amdgcn_sched_barrier(0);       // in this order: hoisted together the reads do not fit the registers
    }
    if (step < a.k) {
      put(lds + (step & 1) * Y_LDS, acc, p);   // read last before the previous barrier
      lds_barrier();
    }
  }
  if (a.G) {
    float* gc = a.G + blk + (i64)(32 * w + 4 * h) * LB + 32 * ct + n;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int r = 8 * (v >> 2) + (v & 3);
      gc[r * LB] = acc[v] + (w == ct && r + 4 * h == n ? 1.f : 0.f);
    }
  }
  if (a.E) {
    // The pair leaves through 2 KB of the buffer that the last product did not read, row by row: 64 bytes of 16 rows per store.
    // Rows of 32 elements in 16-byte chunks, XORed by the row (writes of one column, reads of 16 rows).
    uint16_t* st = reinterpret_cast<uint16_t*>(lds + (a.k & 1) * Y_LDS) + w * 1024;
    uint16_t* e0 = a.E + 2 * blk;
    const int r = lane >> 2, ch = lane & 3;
    auto out = [&](uint16_t* at) {           // at: the tile's first element
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int row = r + 16 * i;
        *reinterpret_cast<u32x4*>(at + row * LB + 8 * ch) = *reinterpret_cast<const u32x4*>(st + row * 32 + 8 * (ch ^ ((row >> 2) & 3)));
      }
    };
#pragma unroll
    for (int v = 0; v < 16; v += 2) {
      const uint32_t pk = mm::pack2_bf16(acc[v], acc[v + 1]);
      const int row = 8 * (v >> 2) + 4 * h + (v & 3);
      const int at = 8 * ((n >> 3) ^ ((row >> 2) & 3)) + (n & 7);       // the same for row + 1
      st[row * 32 + at] = (uint16_t)pk;
      st[(row + 1) * 32 + at] = (uint16_t)(pk >> 16);
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the wave's own writes
    out(e0 + 32 * w * LB + 32 * ct);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // read back before the area is rewritten
#pragma unroll
    for (int g = 0; g < 4; ++g)
      *reinterpret_cast<uint2*>(st + n * 32 + 8 * (g ^ ((n >> 2) & 3)) + 4 * h) =
          make_uint2(mm::pack2_bf16(acc[4 * g], acc[4 * g + 1]), mm::pack2_bf16(acc[4 * g + 2], acc[4 * g + 3]));
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    out(e0 + (i64)LB * LB + 32 * ct * LB + 32 * w);
  }
}

// ---- backward
struct BwdArgs {
  const uint16_t* Tf;      // bf16(T), bf16(D) of all blocks as fragments
  const uint16_t* Df;
  const float* theta[2];   // packed parameters and dL/dG [blocks][LB][LB]: blocks 0 .. nb0 - 1 are the first side's, the rest the second's
  const float* D[2];
  int nb0, k, nb;
  float* dQ;               // dL/dQ [block][row tile][column tile][1024]: tiles in accumulator order
};

// Two waves per SIMD: the fragments of two factors, five tiles in fp32 and what is in flight are some 240 registers.
__global__ __launch_bounds__(512, 2) void cnp_bwd_kernel(BwdArgs a) {
  __shared__ __attribute__((aligned(16))) char lds[4 * Y_LDS];     // U, U', Z, Z'
  const Place p = place();
  if (p.j >= a.nb) return;
  const int lane = p.lane, n = p.n, h = p.h, w = p.w, ct = p.ct;
  const bool second = p.j >= a.nb0;
  const i64 js = second ? p.j - a.nb0 : p.j;
  const bf16x8* tf = reinterpret_cast<const bf16x8*>(a.Tf + (i64)p.j * LB * LB) + lane;
  const bf16x8* df = reinterpret_cast<const bf16x8*>(a.Df + (i64)p.j * LB * LB) + lane;
  bf16x8 AT[NKS], AD[NKS];
  floatx16 T, D, U, Z;         // fp32 tiles (w, ct)
#pragma unroll
  for (int s = 0; s < NKS; ++s) AT[s] = tf[(w * NKS + s) * 64];
  {
    const float* d = (second ? a.D[1] : a.D[0]) + js * LB * LB + (32 * w + 4 * h) * LB + 32 * ct + n;
#pragma unroll
    for (int v = 0; v < 16; ++v) D[v] = d[(8 * (v >> 2) + (v & 3)) * LB];
  }
#pragma unroll
  for (int s = 0; s < NKS; ++s) AD[s] = df[(w * NKS + s) * 64];
  q_tile(T, (second ? a.theta[1] : a.theta[0]) + js * (LB * (LB - 1) / 2), p, -1.f);
  // column n of T as row n of the stripe's own tile (T[k][c] = -T[c][k]): same slots
#pragma unroll
  for (int u = 0; u < 2; ++u)
    *reinterpret_cast<bf16x8*>(lds + (2 * w + u) * 1024 + lane * 16) = negate(tf[(ct * NKS + 2 * w + u) * 64]);
  put(lds + 2 * Y_LDS, D, p);
  U = T;
  Z = D;
  lds_barrier();

  // Z = C + D U_m + T Z_{m-1}; before the last step also the next U = T + T U_m
  auto step = [&](int m, const floatx16& C, floatx16& next, auto LAST) {
    constexpr bool last = decltype(LAST)::value;
    const char* yu = lds + ((m - 1) & 1) * Y_LDS;
    const char* yz = yu + 2 * Y_LDS;
    constexpr int DEPTH = 2;
    bf16x8 fu[DEPTH], fz[DEPTH];
#pragma unroll
    for (int s = 0; s < DEPTH; ++s) {
      fu[s] = fragment(yu, s, lane);
      fz[s] = fragment(yz, s, lane);
    }
#pragma unroll
    for (int s = 0; s < NKS; ++s) {
      const bf16x8 bu = fu[s % DEPTH], bz = fz[s % DEPTH];
      Z = __builtin_amdgcn_mfma_f32_32x32x16_bf16(AD[s], bu, s == 0 ? C : Z, 0, 0, 0);
      if (!last) next = __builtin_amdgcn_mfma_f32_32x32x16_bf16(AT[s], bu, s == 0 ? T : next, 0, 0, 0);
      Z = __builtin_amdgcn_mfma_f32_32x32x16_bf16(AT[s], bz, Z, 0, 0, 0);
      if (s + DEPTH < NKS) {
        fu[s % DEPTH] = fragment(yu, s + DEPTH, lane);
        fz[s % DEPTH] = fragment(yz, s + DEPTH, lane);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  for (int m = 1; m < a.k; ++m) {
    floatx16 next;
    step(m, D, next, std::false_type{});
    floatx16 r = next;
    if (m + 1 == a.k) {
      // U_{k-1} and U_k differ by T^k only and would be rounded to the same bf16 nearly everywhere, so that their errors add up in
      // Z_k + Z_{k-1}: the last one is rounded from where the one before erred to the other side (gradient error at k = 5 2.6e-4 -> 2.3e-4)
#pragma unroll
      for (int v = 0; v < 16; ++v) r[v] -= bf16_bits_to_float((uint16_t)mm::pack2_bf16(U[v], 0.f)) - U[v];
    }
    char* y = lds + (m & 1) * Y_LDS;           // read last before the previous barrier
    put(y, r, p);
    put(y + 2 * Y_LDS, Z, p);
    U = next;
    lds_barrier();
  }
  D += Z;                                      // Z_{k-1}, fp32 as it is in the accumulators
  step(a.k, D, U, std::true_type{});
  float* q = a.dQ + (i64)p.j * LB * LB + (w * NT + ct) * 1024 + lane * 4;
#pragma unroll
  for (int g = 0; g < 4; ++g) *reinterpret_cast<f32x4*>(q + g * 256) = f32x4{Z[4 * g], Z[4 * g + 1], Z[4 * g + 2], Z[4 * g + 3]};
}

inline dim3 chain_grid(int nb) { return dim3((unsigned)ceil_div(nb, 8) * 64); }

}  // namespace

bool lds_cnp_supported(int d, int b) { return b == LB && d % LB == 0; }

void lds_cnp_build(const float* theta, int nb, int k, float* G_f32, void* E_bf16, float* ws, hipStream_t st) {
  uint16_t* Qf = (uint16_t*)ws;
  skew_materialize_chain_launch(theta, nb, nullptr, 0, Qf, nullptr, nullptr, nullptr, st);
  hipLaunchKernelGGL(cnp_build_kernel, chain_grid(nb), dim3(512), 0, st, BuildArgs{Qf, theta, k, nb, G_f32, (uint16_t*)E_bf16});
}

void lds_cnp_bwd(const SeriesSide* sides, int nsides, int k, int accumulate, float* ws, hipStream_t st) {
  const bool two = nsides > 1;
  const int nb0 = sides[0].d / LB, nb1 = two ? sides[1].d / LB : 0, nb = nb0 + nb1;
  const size_t total = (size_t)nb * LB * LB;
  float* dQ = ws;
  uint16_t* Tf = (uint16_t*)(dQ + total);
  uint16_t* Df = Tf + total;
  const SeriesSide& s1 = sides[two ? 1 : 0];
  skew_materialize_chain_launch(sides[0].theta, nb0, s1.theta, nb1, Tf, sides[0].dG, s1.dG, Df, st);
  hipLaunchKernelGGL(cnp_bwd_kernel, chain_grid(nb), dim3(512), 0, st,
                     BwdArgs{Tf, Df, {sides[0].theta, s1.theta}, {sides[0].dG, s1.dG}, nb0, k, nb, dQ});
  skew_project_chain_launch(dQ, nb0, sides[0].dtheta, nb1, s1.dtheta, accumulate, st);
}

}  // namespace poetx
