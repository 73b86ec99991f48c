// Cayley-Neumann series and its backward for b = 256 on chip (Sec. 3.4, Eq. 8-9): one launch runs the whole chain of a
// block's column stripe.
//
// Every quantity of the series is a polynomial in Q applied from the left to a matrix whose
// column stripes do not mix:
//   forward    H_1 = Q,    H_{s+1} = 2Q + Q H_s,       G = I + H_{k+1}
//   backward   R_0 = D^T,  R_m = D^T + Q R_{m-1}        (D = dL/dG)        pass 1, R_m stored
//              Z_0 = D,    Z_m = R_m^T - Q Z_{m-1},     dL/dQ = Z_k + Z_{k-1}   pass 2
// (With T = Q^T = -Q and P_m = sum_{j<=m} D T^j = R_m^T: dL/dQ = sum_p c_p sum_{i+j=p-1} T^i D T^j with c = 2, .., 2, 1
// = P_k + (I + T) sum_{i<k} T^i P_{k-1-i} = Z_k + Z_{k-1}.  Unit coefficients: every step is one product plus a constant,
// which enters as the C operand of the matrix instructions and costs nothing; both passes take k products.)
//
// A workgroup owns 32 columns of a block, its eight waves 32 rows each.  A wave keeps its rows of bf16(Q) in registers as
// matrix-core fragments for the whole chain (64 of them); what moves from step to step is the 256 x 32 stripe of the running matrix, 16 KB
// of bf16 through LDS, two buffers and one barrier per step.  All three chains multiply with the contraction index permuted inside
// groups of 16 (k = 16s + 8a + 4h + j at fragment slot 8h + 4a + j): registers 8u .. 8u + 7 of an accumulator tile then ARE a
// fragment of the next product, so the stripe is written as whole fragments and read back as they lie.  In pass 2 the operands
// are swapped, which leaves the accumulator tile transposed: R_m^T enters it as pass 1 stored R_m, register by register, and
// nothing is transposed on the way; its stripe goes through LDS row by row and comes back with transposing reads.
//
// What bounds it: up to 32 blocks (256 workgroups, one per CU) latency: 4 us of launch, Q and first term, then 0.6 - 0.9 us a step, of
// which 1024 cycles are matrix instructions; for many blocks the traffic of E, R_m and dQ.  Two workgroups fit a CU.  k = 5, us per launch
// (forward / pass 1 / pass 2), with all of Q in LDS and 128 columns in the registers of four waves -> so: 32 blocks 22 / 28 / 30 -> 9.9 / 12 / 12,
// 128 blocks (pass 1 / pass 2) 41 / 43 -> 42 / 41 (R_m at 4 TB/s), 320 blocks forward 84 -> 63.  The forward takes its 2Q from theta itself:
// materialised in fp32 it cost 16 us of 320 blocks' 36.
//
// Precision as in the tiled kernels: products in bf16 with fp32 accumulation, the dominant
// terms (2Q, D, R_m) enter in fp32.
#include "mfma_gemm.h"

namespace poetx {
namespace {

using mm::bf16x8;
using mm::floatx16;
using mm::short4v;
using mm::short8v;

constexpr int LB = 256;                  // block side
constexpr int NT = LB / 32;              // row tiles = waves = column stripes
constexpr int NKS = LB / 16;             // k steps of a product
constexpr int Y_LDS = LB * 32 * 2;       // a stripe of the running matrix

enum { CHAIN_FWD = 0, CHAIN_BWD1 = 1, CHAIN_BWD2 = 2 };

struct ChainArgs {
  const uint16_t* Qf;      // bf16(Q) of all blocks as fragments: [block][row tile][k step][lane][8]
  const float* theta;      // forward
  const float* D[2];       // backward: dL/dG [blocks][LB][LB]; blocks 0 .. nb0 - 1 come from the first side, the rest from the second
  int nb0, j0;             // j0: first block of this launch
  int k, nb;               // nb: blocks of this launch
  float* G;                // forward: I + H, [nb][LB][LB] (nullable)
  uint16_t* E;             // forward: bf16 pair [nb][2][LB][LB] (nullable)
  float* M;                // backward: [k][nb][row tile][column tile][1024]: tiles of R_m in accumulator order
  float* dQ;               // backward pass 2: dL/dQ [all blocks][row tile][column tile][1024], tiles in accumulator order of their transpose
};

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

// this wave's LDS accesses have been carried out, and every other wave's: not __syncthreads(), which would wait for the stores
// of R_m and the loads of the next one as well
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

template <int MODE>
__device__ __forceinline__ void chain(const ChainArgs& a, const int id, char* lds) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);        // this wave's row tile
  // the eight stripes of a block have ids 8 apart: one XCD, whose L2 brings the block's Q in once
  const int j = (id >> 6) * 8 + (id & 7), ct = (id >> 3) & 7;    // block of this launch, column stripe
  if (j >= a.nb) return;
  const int ja = a.j0 + j;                                       // block of all
  const int n = lane & 31, h = lane >> 5;
  const bool second = ja >= a.nb0;
  const i64 js = second ? ja - a.nb0 : ja;

  bf16x8 A[NKS];
  const bf16x8* qf = reinterpret_cast<const bf16x8*>(a.Qf + (i64)ja * LB * LB) + lane;
#pragma unroll
  for (int s = 0; s < NKS; ++s) A[s] = qf[(w * NKS + s) * 64];

  floatx16 acc, C;      // C: the step's fp32 term
  // four consecutive floats per register group; p: the lane's first
  auto load_groups = [&](floatx16& v, const float* p, int stride) {
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const f32x4_a4 x = *reinterpret_cast<const f32x4_a4*>(p + g * stride);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[4 * g + e] = x[e];
    }
  };
  auto store_groups = [&](float* p, const floatx16& v) {
#pragma unroll
    for (int g = 0; g < 4; ++g) *reinterpret_cast<f32x4*>(p + g * 256) = f32x4{v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3]};
  };
  // pass 2: tile (ct, w) of R_m is tile (w, ct) of R_m^T
  auto fetch_r = [&](int step) { load_groups(C, a.M + ((i64)(step - 1) * a.nb + j) * LB * LB + (ct * NT + w) * 1024 + lane * 4, 256); };

  // ---- the fp32 term of the first step and the first running matrix
  if constexpr (MODE == CHAIN_FWD) {
    // lane (n, h), register 4g + e of tile (w, ct): element (i, c) = (32w + 8g + 4h + e, 32ct + n) of 2Q, from the packed triangle
    const float* th = a.theta + (i64)ja * (LB * (LB - 1) / 2);
    const int c = 32 * ct + n, i0 = 32 * w + 4 * h;
    if (w > ct) {          // below the diagonal: minus the mirror image, whose packed row runs along i
      load_groups(C, th + (c * LB - c * (c + 1) / 2 - c - 1) + i0, 8);
#pragma unroll
      for (int v = 0; v < 16; ++v) C[v] *= -2.f;
    } else {
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int i = i0 + 8 * (v >> 2) + (v & 3), lo = i < c ? i : c, hi = i < c ? c : i;   // hi - lo - 1 = -1 on the diagonal: not read
        const float t = lo < hi ? th[lo * LB - lo * (lo + 1) / 2 + hi - lo - 1] : 0.f;
        C[v] = i < c ? 2.f * t : -2.f * t;
      }
    }
    // column n of Q as row n of the stripe's own tile (Q[k][c] = -Q[c][k]): same slots
#pragma unroll
    for (int u = 0; u < 2; ++u)
      *reinterpret_cast<bf16x8*>(lds + (2 * w + u) * 1024 + lane * 16) = negate(qf[(ct * NKS + 2 * w + u) * 64]);
  } else {
    const float* D = (second ? a.D[1] : a.D[0]) + js * LB * LB;
    if constexpr (MODE == CHAIN_BWD1) {        // D^T (w, ct): lane n holds row 32ct + n of D
      load_groups(C, D + (32 * ct + n) * LB + 32 * w + 4 * h, 8);
    } else {                                   // transposed tile: lane n holds row 32w + n of D
      load_groups(acc, D + (32 * w + n) * LB + 32 * ct + 4 * h, 8);
      fetch_r(1);
    }
  }

  // the stripe in LDS.  Natural: fragments [k step][lane].  Transposed tiles: rows of 32 elements, 8-byte pieces XORed by the row / 4.
  const int zrow = 32 * w + n, zf = (n >> 2) & 7;
  auto put = [&](const floatx16& v, char* y) {
    if constexpr (MODE != CHAIN_BWD2) {
#pragma unroll
      for (int u = 0; u < 2; ++u) *reinterpret_cast<bf16x8*>(y + (2 * w + u) * 1024 + lane * 16) = pack8(v, u);
    } else {
#pragma unroll
      for (int g = 0; g < 4; ++g)              // the running matrix is carried negated
        *reinterpret_cast<uint2*>(y + zrow * 64 + 8 * ((2 * g + h) ^ zf)) =
            make_uint2(mm::pack2_bf16(-v[4 * g], -v[4 * g + 1]), mm::pack2_bf16(-v[4 * g + 2], -v[4 * g + 3]));
    }
  };
  // transposing reads: 16 lanes take 4 rows x 32 bytes; rows 16s + 4h .. + 3, then 16s + 8 + 4h .. + 3
  const int ti = lane & 15, tp = 4 * ((lane >> 4) & 1) + (ti & 3);
  const int t_lo = (4 * h + (ti >> 2)) * 64 + 8 * (tp ^ h), t_hi = (8 + 4 * h + (ti >> 2)) * 64 + 8 * (tp ^ (2 + h));
  auto fragment = [&](const char* y, int s) -> bf16x8 {
    if constexpr (MODE != CHAIN_BWD2) return *reinterpret_cast<const bf16x8*>(y + s * 1024 + lane * 16);
    const short4v lo = mm::lds_read_tr(y + s * 1024 + (t_lo ^ (32 * (s & 1)))), hi = mm::lds_read_tr(y + s * 1024 + (t_hi ^ (32 * (s & 1))));
    const short8v v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8, v);
  };
  if constexpr (MODE == CHAIN_BWD1) put(C, lds);
  if constexpr (MODE == CHAIN_BWD2) put(acc, lds);
  lds_barrier();

  // acc = C + Q * running matrix, DEPTH fragments of the stripe in flight.  `after_first` runs once C has been consumed.
  constexpr int DEPTH = MODE == CHAIN_BWD2 ? 2 : 4;   // the registers of four waves per SIMD
  auto product = [&](const char* y, auto after_first) {
    bf16x8 f[DEPTH];
#pragma unroll
    for (int s = 0; s < DEPTH; ++s) f[s] = fragment(y, s);
#pragma unroll
    for (int s = 0; s < NKS; ++s) {
      if constexpr (MODE != CHAIN_BWD2) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[s], f[s % DEPTH], s == 0 ? C : acc, 0, 0, 0);
      else acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[s % DEPTH], A[s], s == 0 ? C : acc, 0, 0, 0);
      if (s + DEPTH < NKS) f[s % DEPTH] = fragment(y, s + DEPTH);
      if (s == 0) after_first();
      __builtin_amdgcn_sched_barrier(0);       // in this order: hoisted together the reads do not fit the registers
    }
  };
  auto nothing = [] {};

  if constexpr (MODE == CHAIN_FWD) {
    for (int step = 1; step <= a.k; ++step) {
      product(lds + ((step - 1) & 1) * Y_LDS, nothing);
      if (step < a.k) {
        put(acc, lds + (step & 1) * Y_LDS);    // read last before the previous barrier
        lds_barrier();
      }
    }
    const i64 blk = (i64)ja * LB * LB;
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
  } else if constexpr (MODE == CHAIN_BWD1) {
    for (int step = 1; step <= a.k; ++step) {
      product(lds + ((step - 1) & 1) * Y_LDS, nothing);
      if (step < a.k) put(acc, lds + (step & 1) * Y_LDS);
      store_groups(a.M + ((i64)(step - 1) * a.nb + j) * LB * LB + (w * NT + ct) * 1024 + lane * 4, acc);
      if (step < a.k) lds_barrier();
    }
  } else {
    int step = 1;
    do {
      if (step == a.k) C += acc;               // the last one carries Z_{k-1} (fp32, still in the accumulators) into the sum
      product(lds + ((step - 1) & 1) * Y_LDS, [&] { if (step < a.k) fetch_r(step + 1); });
      put(acc, lds + (step & 1) * Y_LDS);
      lds_barrier();
    } while (++step <= a.k);
    store_groups(a.dQ + (i64)ja * LB * LB + (w * NT + ct) * 1024 + lane * 4, acc);
  }
}

template <int MODE>
__global__ __launch_bounds__(512, 4) void cnp_chain_kernel(ChainArgs a) {
  __shared__ __attribute__((aligned(16))) char lds[2 * Y_LDS];
  chain<MODE>(a, blockIdx.x, lds);
}
template <int MODE>
void launch_chain(const ChainArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(cnp_chain_kernel<MODE>, dim3((unsigned)ceil_div(a.nb, 8) * 64), dim3(512), 0, st, a);
}

}  // namespace

bool lds_cnp_supported(int d, int b) { return b == LB && d % LB == 0; }

void lds_cnp_build(const float* theta, int nb, int k, float* G_f32, void* E_bf16, float* ws, hipStream_t st) {
  uint16_t* Qf = (uint16_t*)ws;
  skew_materialize_chain_launch(theta, nb, nullptr, 0, Qf, st);
  ChainArgs a{};
  a.Qf = Qf;
  a.theta = theta;
  a.nb0 = nb;
  a.k = k;
  a.nb = nb;
  a.G = G_f32;
  a.E = (uint16_t*)E_bf16;
  launch_chain<CHAIN_FWD>(a, st);
}

// Blocks per pair of backward launches, of those left: from 64 on the passes are bound by the R_m between them (k * 256 KB per
// block, written at 4 TB/s), which stay in the 256 MB memory-side cache for up to 128 blocks, being rewritten in place by the next group;
// a remainder goes in halves.  Backward at k = 5, us, 128 a time / 64 / 96 / 136: 200 blocks 166 / 168 / 172 / 164, 320: 247 / 255 / 257 / 263;
// 160 as 128 + 32 135, as 96 + 64 124; 144 at once 122, as 96 + 48 113.
constexpr int GROUP_MOST = 128;
inline int group_size(int left) { return left <= GROUP_MOST ? left : left < 192 ? (left + 15) / 16 * 8 : GROUP_MOST; }
inline int max_group(int blocks) { return blocks < GROUP_MOST ? blocks : GROUP_MOST; }   // bound on any group's size

size_t lds_cnp_bwd_ws_floats(int nb, int k) {
  const size_t bb = (size_t)LB * LB;
  return ((size_t)k * max_group(nb) + nb) * bb + nb * bb / 2;
}

void lds_cnp_bwd(const SeriesSide* sides, int nsides, int k, int accumulate, float* ws, hipStream_t st) {
  ChainArgs a{};
  int nb = 0;
  for (int i = 0; i < nsides; ++i) {
    a.D[i] = sides[i].dG;
    nb += sides[i].d / LB;
  }
  a.nb0 = sides[0].d / LB;
  a.k = k;
  a.dQ = ws;
  a.M = ws + (size_t)nb * LB * LB;
  uint16_t* Qf = (uint16_t*)(a.M + (size_t)k * max_group(nb) * LB * LB);
  skew_materialize_chain_launch(sides[0].theta, a.nb0, nsides > 1 ? sides[1].theta : nullptr, nb - a.nb0, Qf, st);
  a.Qf = Qf;
  for (a.j0 = 0; a.j0 < nb; a.j0 += a.nb) {
    a.nb = group_size(nb - a.j0);
    launch_chain<CHAIN_BWD1>(a, st);
    launch_chain<CHAIN_BWD2>(a, st);
  }
  skew_project_chain_launch(a.dQ, a.nb0, sides[0].dtheta, nb - a.nb0, nsides > 1 ? sides[1].dtheta : nullptr, accumulate, st);
}

}  // namespace poetx
