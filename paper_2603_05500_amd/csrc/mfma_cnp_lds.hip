// Cayley-Neumann series and its backward for b = 256 with the block resident on chip
// (Sec. 3.4, Eq. 8-9): one launch runs the whole chain of a block.
//
// Every quantity of the series is a polynomial in Q applied from the left to a matrix whose
// column stripes do not mix:
//   forward    H_1 = Q,    H_{s+1} = 2Q + Q H_s,       G = I + H_{k+1}
//   backward   R_0 = D^T,  R_m = D^T + Q R_{m-1}        (D = dL/dG)        pass 1, R_m stored
//              Z_0 = D,    Z_m = R_m^T - Q Z_{m-1},     dL/dQ = Z_k + Z_{k-1}   pass 2
// (With T = Q^T = -Q and P_m = sum_{j<=m} D T^j = R_m^T: dL/dQ = sum_p c_p sum_{i+j=p-1} T^i D T^j with c = 2, .., 2, 1
// = P_k + (I + T) sum_{i<k} T^i P_{k-1-i} = Z_k + Z_{k-1}.  Unit coefficients: every step is one product plus a constant,
// which enters as the C operand of the matrix instructions and costs nothing; both passes take k products.)
// So one kernel serves all three: bf16(Q) (materialised once per call from the packed parameters by a small kernel that
// spreads over the whole chip; building it in LDS here, in three different ways, cost 16 us per launch in serial
// latencies) sits in LDS as the left operand, a wave owns 32 columns of the running matrix and keeps them in registers as
// matrix-core B fragments, multiplies (v_mfma_f32_32x32x16_bf16, fp32 accumulators that start from the step's fp32 term,
// 8 row tiles) and rounds the result straight back into B fragments: with the
// contraction index permuted inside each group of 16 (k = 16s + 8a + 4h + j is taken at
// fragment slot 8h + 4a + j) accumulator registers 8u..8u+7 of row tile t ARE fragment
// 2t+u, so the chain never leaves the register file and nothing is transposed.  The same
// permutation is applied to the columns of Q in LDS, which keeps its fragment reads 16 bytes
// wide.  A workgroup is 4 waves = 128 columns; two workgroups share a block.
//
// What bounds it: a product is 4100 cycles of matrix instructions and as many of LDS fragment reads, and everything else
// of a launch is latency and address processing on few waves.  Hence every 32 x 32 tile that enters or leaves goes
// through a per-wave LDS area, so that all global accesses are 16 bytes per lane on whole 128-byte lines (written from the
// accumulator layout, 32 scattered 16-byte pieces per instruction, the R_m of a step took twice the time of its
// product), and R_m is stored tile by tile in the order in which pass 2 loads it.  Cycles of a workgroup at k = 5
// (32 blocks): forward 61 -> 45 thousand, pass 1 76 -> 57, pass 2 59 -> 60 (with scalar loads of D and of the W it used to read);
// a step is 5.7 / 8.9 / 8.2 thousand.
//
// Precision as in the tiled kernels: products in bf16 with fp32 accumulation, the dominant
// terms (2Q, D, R_m) enter in fp32.
#include "mfma_gemm.h"

namespace poetx {
namespace {

using mm::bf16x8;
using mm::floatx16;

constexpr int LB = 256;                  // block side
constexpr int LROW = LB * 2 + 16;        // LDS row stride in bytes: 16 lanes of a 16-byte read hit 16 bank groups
constexpr int Q_LDS = LB * LROW;         // 135168 bytes
constexpr int TLD = 36;                  // row stride (floats) of a staged 32 x 32 fp32 tile: 16-byte pieces, banks spread
constexpr int STG_LDS = 32 * TLD * 4;    // staging of a wave
constexpr int CHAIN_LDS = Q_LDS + 4 * STG_LDS;   // 153600 bytes
constexpr int NT = LB / 32;              // row tiles of a stripe
constexpr int NKS = LB / 16;             // k steps of a product

enum { CHAIN_FWD = 0, CHAIN_BWD1 = 1, CHAIN_BWD2 = 2 };

struct ChainArgs {
  const uint16_t* Qb;      // bf16(Q) of all blocks, [nb][LB][LB] row major
  const float* Q2;         // forward: 2Q in fp32, [nb][column tile][row tile][1024], tiles in accumulator order
  const float* D[2];       // backward: dL/dG [blocks][LB][LB]; blocks 0 .. nb0 - 1 come from the first side, the rest from the second
  int nb0, j0;             // j0: first block of this launch
  int k, nb;               // nb: blocks of this launch
  float* G;                // forward: I + H, [nb][LB][LB] (nullable)
  uint16_t* E;             // forward: bf16 pair [nb][2][LB][LB] (nullable)
  float* M;                // backward: [k][nb][tile a][tile b][1024]: tile (a, b) of R_m, transposed, in accumulator order
  float* dQ;               // backward pass 2: dL/dQ [all blocks][LB][LB]
};

// p + n with the sum hidden from the optimiser: walking a column row by row with this keeps
// one live address instead of one precomputed 64-bit address per unrolled access.  The pointer carries the global
// address space -- behind the asm the compiler cannot infer it, and a flat access would count as an LDS one too and make
// every fragment read wait for it.
template <class T>
using glob = __attribute__((address_space(1))) T*;
template <class T>
__device__ inline glob<T> bump(glob<T> p, i64 n) {
  p += n;
  asm volatile("" : "+v"(p));
  return p;
}

__device__ inline bf16x8 negate(bf16x8 v) {
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  u32x4 u = __builtin_bit_cast(u32x4, v);
  u ^= 0x80008000u;
  return __builtin_bit_cast(bf16x8, u);
}

template <bool NEG>
__device__ inline bf16x8 pack8(const floatx16& a, int u) {
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  u32x4 r;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float x = a[8 * u + 2 * e], y = a[8 * u + 2 * e + 1];
    r[e] = NEG ? mm::pack2_bf16(-x, -y) : mm::pack2_bf16(x, y);
  }
  return __builtin_bit_cast(bf16x8, r);
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// bf16(Q) of a block into LDS, contraction slots permuted: a 16-byte chunk (8 consecutive k, i.e. one value of a and both
// values of h) becomes two 8-byte pieces 16 bytes apart.
constexpr int NCH = LB * LB / 8 / 256;   // chunks per thread
// Chunk (row, kc) of a wave's two rows goes to lane 16 * (2 * (kc >> 4) + (row & 1)) + (kc & 15): the 8-byte
// writes of a half wave then cover rows 2p and 2p + 1 (4 banks apart) over 16 chunks each = all 64 banks once.
__device__ __forceinline__ void chunk_of(int id, int& row, int& kc) {
  const int l = id & 63;
  row = 2 * (id >> 6) + ((l >> 4) & 1);
  kc = (l & 15) + 16 * (l >> 5);
}
__device__ __forceinline__ void fetch_q(u32x4 (&v)[NCH], const uint16_t* Qb, int tid) {
  const u32x4* src = reinterpret_cast<const u32x4*>(Qb);
#pragma unroll
  for (int it = 0; it < NCH; ++it) {
    int row, kc;
    chunk_of(tid + 256 * it, row, kc);
    v[it] = src[row * 32 + kc];
  }
}
__device__ __forceinline__ void store_q(char* lds, const u32x4 (&v)[NCH], int tid) {
#pragma unroll
  for (int it = 0; it < NCH; ++it) {
    int row, kc;
    chunk_of(tid + 256 * it, row, kc);
    char* dst = lds + row * LROW + 32 * (kc >> 1) + 8 * (kc & 1);
    *reinterpret_cast<uint2*>(dst) = make_uint2(v[it][0], v[it][1]);
    *reinterpret_cast<uint2*>(dst + 16) = make_uint2(v[it][2], v[it][3]);
  }
}

// ---- 32 x 32 fp32 tiles through the wave's staging area.  A raw tile is what four 16-byte loads per lane bring: piece i
// of lane l is row l / 8 + 8 i, columns 4 (l % 8) .. + 3.  The area is private to the wave, and a wave's LDS instructions
// execute in the order they are issued: keeping the compiler from reordering them is all the synchronisation, and the
// next tile's writes follow this tile's reads without waiting for them.
__device__ __forceinline__ void stage_fence() { asm volatile("" ::: "memory"); }
__device__ __forceinline__ void stage_raw(float* stg, const floatx16& raw, int lane) {
#pragma unroll
  for (int i = 0; i < 4; ++i)
    *reinterpret_cast<f32x4*>(stg + (lane / 8 + 8 * i) * TLD + 4 * (lane % 8)) = f32x4{raw[4 * i], raw[4 * i + 1], raw[4 * i + 2], raw[4 * i + 3]};
  stage_fence();
}
// accumulator layout of the staged tile: lane (n, h), register 4g + e = element (8g + 4h + e, n)
__device__ __forceinline__ void unstage(const float* stg, floatx16& v, int n, int h) {
#pragma unroll
  for (int g = 0; g < 4; ++g)
#pragma unroll
    for (int e = 0; e < 4; ++e) v[4 * g + e] = stg[(8 * g + 4 * h + e) * TLD + n];
  stage_fence();
}
// ... of its transpose: element (n, 8g + 4h + e)
__device__ __forceinline__ void unstage_t(const float* stg, floatx16& v, int n, int h) {
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const f32x4 x = *reinterpret_cast<const f32x4*>(stg + n * TLD + 8 * g + 4 * h);
#pragma unroll
    for (int e = 0; e < 4; ++e) v[4 * g + e] = x[e];
  }
  stage_fence();
}

template <int MODE>
__global__ __launch_bounds__(256) void cnp_chain_kernel(ChainArgs a) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j = blockIdx.y;                     // block of this launch
  const int ja = a.j0 + j;                      // of all
  const int n = lane & 31, h = lane >> 5;
  const int ct = blockIdx.x * 4 + wave;         // this wave's column tile
  const int col = ct * 32 + n;                  // this lane's column of the running matrix
  const i64 blk = (i64)ja * LB * LB;
  const bool second = ja >= a.nb0;
  const i64 js = second ? ja - a.nb0 : ja;
  float* stg = reinterpret_cast<float*>(lds + Q_LDS) + wave * (STG_LDS / 4);

  bf16x8 Y[NKS];
  floatx16 acc[NT], C[NT];      // C: the step's fp32 term
  u32x4 qv[NCH];
  fetch_q(qv, a.Qb + blk, tid);
  // the fp32 term's raw tiles are in flight with Q and land under its way into LDS
  const int lr = lane / 8, lc = 4 * (lane % 8);
  auto raw_tile = [&](floatx16& v, const float* p) {   // p: the lane's first element of a tile with rows of LB
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const f32x4 x = *reinterpret_cast<const f32x4*>(p + 8 * i * LB);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[4 * i + e] = x[e];
    }
  };
  // pass 2: R_m^T (t, ct) is tile (ct, t) of R_m, transposed
  auto fetch_r = [&](int step) {
    const float* in = a.M + ((i64)(step - 1) * a.nb + j) * LB * LB + ct * (NT * 1024) + lane * 4;
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const f32x4 x = *reinterpret_cast<const f32x4*>(in + t * 1024 + g * 256);
#pragma unroll
        for (int e = 0; e < 4; ++e) C[t][4 * g + e] = x[e];
      }
  };
  if constexpr (MODE == CHAIN_FWD) {
    const float* q2 = a.Q2 + blk + ct * (NT * 1024) + lane * 4;   // 2Q, already in accumulator order
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const f32x4 x = *reinterpret_cast<const f32x4*>(q2 + t * 1024 + g * 256);
#pragma unroll
        for (int e = 0; e < 4; ++e) C[t][4 * g + e] = x[e];
      }
  } else {
    const float* D = (second ? a.D[1] : a.D[0]) + js * LB * LB;
    if constexpr (MODE == CHAIN_BWD1) {   // D^T (t, ct) = transpose of D (ct, t)
#pragma unroll
      for (int t = 0; t < NT; ++t) raw_tile(C[t], D + (32 * ct + lr) * LB + 32 * t + lc);
    } else {
#pragma unroll
      for (int t = 0; t < NT; ++t) raw_tile(acc[t], D + (32 * t + lr) * LB + 32 * ct + lc);
    }
  }

  store_q(lds, qv, tid);
  __syncthreads();

  // A fragment (row tile tm, k step s): 16 bytes at row 32 tm + n, slot 16 s + 8 h.
  const char* qa = lds + n * LROW + 16 * h;

  // ---- first value of the running matrix, the fp32 term in accumulator layout
  if constexpr (MODE == CHAIN_FWD) {
    // the lane's own column of Q read as row `col` (Q[k][col] = -Q[col][k]): same slots
    const char* qown = lds + col * LROW + 16 * h;
#pragma unroll
    for (int s = 0; s < NKS; ++s) Y[s] = negate(*reinterpret_cast<const bf16x8*>(qown + s * 32));
  } else if constexpr (MODE == CHAIN_BWD1) {
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      stage_raw(stg, C[t], lane);
      unstage_t(stg, C[t], n, h);
      Y[2 * t] = pack8<false>(C[t], 0);
      Y[2 * t + 1] = pack8<false>(C[t], 1);
    }
  } else {
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      stage_raw(stg, acc[t], lane);
      unstage(stg, acc[t], n, h);
      Y[2 * t] = pack8<true>(acc[t], 0);     // the running matrix is carried negated
      Y[2 * t + 1] = pack8<true>(acc[t], 1);
    }
  }

  // acc = C + Q * running matrix; the fragments of the next k step are read under the MFMAs of this one.  `after_first`
  // runs once C has been consumed.
  auto product = [&](auto after_first) {
    bf16x8 A[2][NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) A[0][t] = *reinterpret_cast<const bf16x8*>(qa + t * 32 * LROW);
#pragma unroll
    for (int s = 0; s < NKS; ++s) {
      if (s + 1 < NKS) {
#pragma unroll
        for (int t = 0; t < NT; ++t)
          A[(s + 1) & 1][t] = *reinterpret_cast<const bf16x8*>(qa + t * 32 * LROW + (s + 1) * 32);
      }
#pragma unroll
      for (int t = 0; t < NT; ++t)
        acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[s & 1][t], Y[s], s == 0 ? C[t] : acc[t], 0, 0, 0);
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
      __builtin_amdgcn_sched_barrier(0);   // keep the reads of step s+1 in the shadow of step s
      if (s == 0) after_first();
    }
  };
  auto nothing = [] {};
  auto repack = [&](auto NEG) {
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      Y[2 * t] = pack8<decltype(NEG)::value>(acc[t], 0);
      Y[2 * t + 1] = pack8<decltype(NEG)::value>(acc[t], 1);
    }
  };

  if constexpr (MODE == CHAIN_FWD) {
    for (int step = 1; step <= a.k; ++step) {
      product(nothing);
      if (step < a.k) repack(std::false_type{});
    }
    if (a.G) {
      glob<float> gc = (glob<float>)(a.G + blk + col + (i64)4 * h * LB);
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
#pragma unroll
          for (int e = 0; e < 4; ++e) gc[e * LB] = acc[t][4 * g + e] + ((32 * t + 8 * g + 4 * h + e) == col ? 1.f : 0.f);
          gc = bump(gc, 8 * LB);
        }
    }
    if (a.E) {
      // The pair leaves through LDS, in Q's place: the wave's 256 x 32 stripe of E with rows of 40 elements, then its
      // transpose with rows of 264.
      constexpr int LE = 40, LT = LB + 8;
      __syncthreads();                           // every wave is done with Q
      uint16_t* st = reinterpret_cast<uint16_t*>(lds) + wave * (LB * LE);
      uint16_t* e0 = a.E + (i64)ja * 2 * LB * LB;
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int v = 0; v < 16; v += 2) {
          const uint32_t pk = mm::pack2_bf16(acc[t][v], acc[t][v + 1]);
          const int r = 32 * t + 8 * (v >> 2) + 4 * h + (v & 3);
          st[r * LE + n] = (uint16_t)pk;
          st[(r + 1) * LE + n] = (uint16_t)(pk >> 16);
        }
      stage_fence();
#pragma unroll 8
      for (int i = 0; i < LB / 16; ++i) {        // 4 lanes on a row's 64 bytes
        const int r = 16 * i + lane / 4, c = 8 * (lane % 4);
        *reinterpret_cast<u32x4*>(e0 + r * LB + 32 * ct + c) = *reinterpret_cast<const u32x4*>(st + r * LE + c);
      }
      stage_fence();
      uint16_t* e1 = e0 + (i64)LB * LB + 32 * ct * LB;
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int g = 0; g < 4; ++g)
          *reinterpret_cast<uint2*>(st + n * LT + 32 * t + 8 * g + 4 * h) =
              make_uint2(mm::pack2_bf16(acc[t][4 * g], acc[t][4 * g + 1]), mm::pack2_bf16(acc[t][4 * g + 2], acc[t][4 * g + 3]));
      stage_fence();
#pragma unroll 8
      for (int i = 0; i < 16; ++i) {             // 32 lanes on a row's 512 bytes
        const int r = 2 * i + lane / 32, c = 8 * (lane % 32);
        *reinterpret_cast<u32x4*>(e1 + r * LB + c) = *reinterpret_cast<const u32x4*>(st + r * LT + c);
      }
    }
  } else if constexpr (MODE == CHAIN_BWD1) {
    for (int step = 1; step <= a.k; ++step) {
      product(nothing);
      // tile (t, ct) of R_m leaves transposed, in the order pass 2 loads it
      float* out = a.M + ((i64)(step - 1) * a.nb + j) * LB * LB + ct * 1024 + lane * 4;
      floatx16 v[2];
      auto turn = [&](int t) {
#pragma unroll
        for (int g = 0; g < 4; ++g)
          *reinterpret_cast<f32x4*>(stg + n * TLD + 8 * g + 4 * h) = f32x4{acc[t][4 * g], acc[t][4 * g + 1], acc[t][4 * g + 2], acc[t][4 * g + 3]};
        stage_fence();
        unstage(stg, v[t & 1], n, h);
      };
      turn(0);
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        if (t + 1 < NT) turn(t + 1);             // the next tile is on its way through LDS while this one is stored
#pragma unroll
        for (int g = 0; g < 4; ++g)
          *reinterpret_cast<f32x4*>(out + t * (NT * 1024) + g * 256) = f32x4{v[t & 1][4 * g], v[t & 1][4 * g + 1], v[t & 1][4 * g + 2], v[t & 1][4 * g + 3]};
      }
      if (step < a.k) repack(std::false_type{});
    }
  } else {
    fetch_r(1);                   // the next step's tiles of R are fetched under the product
    for (int step = 1; step <= a.k; ++step) {
      if (step == a.k) {          // the last one carries Z_{k-1} (fp32, still in the accumulators) into the sum
#pragma unroll
        for (int t = 0; t < NT; ++t) C[t] += acc[t];
      }
      product([&] { if (step < a.k) fetch_r(step + 1); });
      if (step < a.k) repack(std::true_type{});
    }
    glob<float> p = (glob<float>)(a.dQ + blk + col + (i64)4 * h * LB);
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
#pragma unroll
        for (int e = 0; e < 4; ++e) p[e * LB] = acc[t][4 * g + e];
        p = bump(p, 8 * LB);
      }
  }
}

template <int MODE>
void launch_chain(const ChainArgs& a, hipStream_t st) {
  auto kern = cnp_chain_kernel<MODE>;
  // once per kernel instance; a function-local static is initialised exactly once, whichever thread gets there first
  static const bool configured =
      hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, CHAIN_LDS) == hipSuccess;
  (void)configured;
  hipLaunchKernelGGL(kern, dim3(LB / 128, a.nb), dim3(256), CHAIN_LDS, st, a);
}

}  // namespace

bool lds_cnp_supported(int d, int b) { return b == LB && d % LB == 0; }

void lds_cnp_build(const float* theta, int nb, int k, float* G_f32, void* E_bf16, float* ws, hipStream_t st) {
  uint16_t* Qb = (uint16_t*)(ws + (size_t)nb * LB * LB);
  skew_materialize_chain_launch(theta, nb, nullptr, 0, ws, Qb, st);
  ChainArgs a{};
  a.Qb = Qb;
  a.Q2 = ws;
  a.nb0 = nb;
  a.k = k;
  a.nb = nb;
  a.G = G_f32;
  a.E = (uint16_t*)E_bf16;
  launch_chain<CHAIN_FWD>(a, st);
}

// Blocks per pair of backward launches, of those left: 128 are two workgroups per block on 256 CUs, once, and the R_m between the two
// passes (k * 256 KB per block) stay in the 256 MB memory-side cache, being rewritten in place by the next group; a short
// remainder joins the last group.  Build + backward at k = 5, all at once / groups of 128, us: 130 blocks 213 / 222, 144: 226 / 224,
// 200: 280 / 260, 320: 438 / 404.
constexpr int GROUP_MOST = 144;
inline int group_size(int left) { return left <= GROUP_MOST ? left : 128; }
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
  uint16_t* Qb = (uint16_t*)(a.M + (size_t)k * max_group(nb) * LB * LB);
  skew_materialize_chain_launch(sides[0].theta, a.nb0, nsides > 1 ? sides[1].theta : nullptr, nb - a.nb0, nullptr, Qb, st);
  a.Qb = Qb;
  for (a.j0 = 0; a.j0 < nb; a.j0 += a.nb) {
    a.nb = group_size(nb - a.j0);
    launch_chain<CHAIN_BWD1>(a, st);
    launch_chain<CHAIN_BWD2>(a, st);
  }
  const float* M = a.dQ;
  skew_project_sides_launch(M, LB, a.nb0, sides[0].dtheta, nb - a.nb0, nsides > 1 ? sides[1].dtheta : nullptr, accumulate, st);
}

}  // namespace poetx
