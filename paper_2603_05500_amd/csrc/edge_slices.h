// Dense product of small and ragged problems whose operands lie on 16-byte boundaries: every wave takes the whole output tile for its own slices
// of the contraction.
//
//   C(i, j) = sum_k A(i, k) * B(k, j)
//
// A slice is 64 bytes of a K-major operand's rows (32 bf16 or 16 fp32 of depth).  Slices w, w + WAVES, ... go to wave w, straight into an LDS ring of
// its own (direct-to-LDS loads, swizzled like the other kernels' tiles), so its own vmcnt is all it ever waits for: no barrier until the
// partial tiles meet in LDS at the end, where all waves add them, each eight columns of a row per lane, in order.
//
// What bounds the edge kernel at these sizes is the chain of a stage: load, wait, LDS store, barrier, with one stage in flight.  Here
// WAVES x NS slices are, and a short contraction is in flight as a whole.
#pragma once
#include "edge_gemm.h"

namespace poetx {
namespace edge {

// at most `slices` (<= MAX, wave uniform) slices of LPS loads each may stay in flight
template <int LPS, int MAX>
__device__ __forceinline__ void wait_slices(int slices) {
  if constexpr (MAX <= 0) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  } else {
    if (slices >= MAX) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(MAX * LPS) : "memory");
    else wait_slices<LPS, MAX - 1>(slices);
  }
}

// slices of a whole contraction (a multiple of a slice's depth).  No product of K and the element size: K goes up to the last int.
constexpr int slice_count(int K, int element) { return K / (64 / element); }
static_assert(slice_count(1 << 29, 4) == 1 << 25 && slice_count(1 << 30, 2) == 1 << 25 && slice_count(0x7fffffe0, 2) == 0x3ffffff, "the bytes of such a row are more than an int holds");

template <class T, int BM, int BN, int WAVES, int NS>
struct SliceShape {
  static constexpr int DEPTH = 64 / (int)sizeof(T);            // of a slice
  static constexpr int NA = BM / 16, NB = BN / 16;             // direct-to-LDS instructions of a slice
  static constexpr int SLICE = (BM + BN) * 64, RING = NS * SLICE;
  static constexpr int LDC = BN + 4, PART = BM * LDC * 4;      // a wave's partial tile, fp32
  static constexpr int TM = BM / 32, TN = BN / 32;
  static constexpr int LDS = WAVES * (RING > PART ? RING : PART);
  static_assert(NS * (NA + NB) < 64, "vmcnt range");
};

// Chunk of the tile (row, 16-byte chunk of it) that lane slot `slot` of an operand's slice holds; its inverse is where a fragment reads.
template <class T, int X, bool K_MAJOR>
__device__ __forceinline__ void slice_chunk(int slot, int& row, int& chunk) {
  constexpr int CPR = K_MAJOR ? 4 : X * (int)sizeof(T) / 16;
  row = slot / CPR;
  const int p = slot % CPR;
  if constexpr (K_MAJOR) chunk = mm::xk_chunk(p, row);
  else if constexpr (sizeof(T) == 2) {
    if constexpr (X >= 64) chunk = mm::kx_unchunk<X>(p, row);
    else chunk = p;
  } else if constexpr (X >= 64) {      // fp32: a fragment reads rows k and k + 4 at once, which must not meet on the banks
    chunk = p ^ (8 * ((row >> 2) & 1));
  } else {
    chunk = p;
    row ^= (row >> 2) & 1;
  }
}
// fp32, X major: float offset of element (k, x)
template <int X>
__device__ __forceinline__ int slice_f32_at(int k, int x) {
  if constexpr (X >= 64) return k * X + (x ^ (32 * ((k >> 2) & 1)));
  else return (k ^ ((k >> 2) & 1)) * X + x;
}

struct SliceArgs {
  const void *A, *B;
  i64 lda, ldb;
  int M, cols;            // rows of A (output rows), columns of B: loads past them fetch the last ones, whose results nobody stores
  int tiles_m, slices;    // slices: of the whole contraction
  int slices_per_split;
};

// two waves per SIMD (256 registers): a second workgroup on the CU hides the first one's ends
template <class T, int BM, int BN, int WAVES, int NS, bool A_K, class Epi>
__global__ __launch_bounds__(64 * WAVES, 2) void slice_kernel(SliceArgs g, Epi epi) {
  using S = SliceShape<T, BM, BN, WAVES, NS>;
  constexpr int V = 16 / (int)sizeof(T), DEPTH = S::DEPTH, NA = S::NA, NB = S::NB, TM = S::TM, TN = S::TN;
  constexpr bool BF = sizeof(T) == 2;
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // each XCD takes a contiguous run of tiles, rows first: they share columns of B
  const int total = gridDim.x, xcd = blockIdx.x & 7, per = total >> 3, extra = total & 7;
  const int id = xcd * per + (xcd < extra ? xcd : extra) + (blockIdx.x >> 3);
  const int i0 = (id % g.tiles_m) * BM, j0 = (id / g.tiles_m) * BN, split = blockIdx.y;
  const int first = split * g.slices_per_split;
  const int count = g.slices - first < g.slices_per_split ? g.slices - first : g.slices_per_split;
  const int mine = (count - wave + WAVES - 1) / WAVES;      // this wave's slices: first + wave, + WAVES, ...

  // per-lane byte offsets from the tile's first element, the same for every slice
  uint32_t voffA[NA], voffB[NB];
#pragma unroll
  for (int s = 0; s < NA; ++s) {
    int r, c;
    slice_chunk<T, BM, A_K>(s * 64 + lane, r, c);
    if (A_K) voffA[s] = (uint32_t)(((i0 + r < g.M ? r : g.M - 1 - i0) * g.lda + c * V) * sizeof(T));
    else voffA[s] = (uint32_t)((r * g.lda + (i0 + c * V < g.M ? c * V : g.M - V - i0)) * sizeof(T));
  }
#pragma unroll
  for (int s = 0; s < NB; ++s) {
    int r, c;
    slice_chunk<T, BN, false>(s * 64 + lane, r, c);
    voffB[s] = (uint32_t)((r * g.ldb + (j0 + c * V < g.cols ? c * V : g.cols - V - j0)) * sizeof(T));
  }
  const T* A0 = (const T*)g.A + (A_K ? i0 * g.lda : (i64)i0);
  const T* B0 = (const T*)g.B + j0;
  char* const ring = lds + wave * S::RING;
  const uint32_t ring_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)ring;
  auto issue = [&](int t) {
    const i64 k = (i64)(first + wave + t * WAVES) * DEPTH;
    const T* a = A0 + (A_K ? k : k * g.lda);
    const T* b = B0 + k * g.ldb;
    const uint32_t at = ring_base + (t % NS) * S::SLICE;
#pragma unroll
    for (int s = 0; s < NA; ++s) asm volatile("global_load_lds_dwordx4 %0, %1" ::"v"(voffA[s]), "s"(a), "{m0}"(at + s * 1024) : "memory");
#pragma unroll
    for (int s = 0; s < NB; ++s) asm volatile("global_load_lds_dwordx4 %0, %1" ::"v"(voffB[s]), "s"(b), "{m0}"(at + (NA + s) * 1024) : "memory");
  };

  // fp32: a wave's slices go to two sums in turn, which halves the chain that rounding errors add up along.  rms error against 64 bits over 120 products, forward, relative to
  // the edge kernel's (which splits deep contractions over workgroups), and the fp32 step of 1024 x 768 with 1001 tokens: one sum 1.15, 80.5 us; two 0.90, 81.2; two of which one is
  // closed every 64 of depth 0.88, 86.0.
  constexpr int SUMS = BF ? 1 : 2;
  typedef floatx16 Acc[TM][TN];
  Acc sums[SUMS];
#pragma unroll
  for (int i = 0; i < SUMS; ++i)
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
      for (int c = 0; c < TN; ++c)
#pragma unroll
        for (int v = 0; v < 16; ++v) sums[i][a][c][v] = 0.f;

  const int li = lane & 31, h = lane >> 5;
  auto multiply = [&](const char* sA, Acc& acc) {
    const char* sB = sA + BM * 64;
    if constexpr (BF) {
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        bf16x8 fa[TM], fb[TN];
#pragma unroll
        for (int a = 0; a < TM; ++a) fa[a] = frag_bf16<BM, A_K>(sA, a * 32, ks);
#pragma unroll
        for (int c = 0; c < TN; ++c) fb[c] = frag_bf16<BN, false>(sB, c * 32, ks);
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
          for (int c = 0; c < TN; ++c) acc[a][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[c], fa[a], acc[a][c], 0, 0, 0);
      }
    } else {
      // a matrix instruction takes two k; lane half h holds k = 8 j + 4 h + e for step e of group j
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        float fa[TM][4], fb[TN][4];
#pragma unroll
        for (int a = 0; a < TM; ++a) {
          if constexpr (A_K) {
            const int r = a * 32 + li;
            const float4 v = *reinterpret_cast<const float4*>(sA + r * 64 + 16 * mm::xk_chunk(2 * j + h, r));
            fa[a][0] = v.x; fa[a][1] = v.y; fa[a][2] = v.z; fa[a][3] = v.w;
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) fa[a][e] = reinterpret_cast<const float*>(sA)[slice_f32_at<BM>(8 * j + 4 * h + e, a * 32 + li)];
          }
        }
#pragma unroll
        for (int c = 0; c < TN; ++c)
#pragma unroll
          for (int e = 0; e < 4; ++e) fb[c][e] = reinterpret_cast<const float*>(sB)[slice_f32_at<BN>(8 * j + 4 * h + e, c * 32 + li)];
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int a = 0; a < TM; ++a)
#pragma unroll
            for (int c = 0; c < TN; ++c) acc[a][c] = __builtin_amdgcn_mfma_f32_32x32x2f32(fb[c][e], fa[a][e], acc[a][c], 0, 0, 0);
      }
    }
  };

#pragma unroll
  for (int t = 0; t < NS; ++t)
    if (t < mine) issue(t);
  auto step = [&](int t, Acc& acc) {
    // slice t has landed: at most the slices issued after it are in flight
    const int younger = mine - 1 - t < NS - 1 ? mine - 1 - t : NS - 1;
    wait_slices<NA + NB, NS - 1>(younger);
    multiply(ring + (t % NS) * S::SLICE, acc);
    if (t + NS < mine) {
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // read before the slot is refilled
      issue(t + NS);
    }
  };
  for (int t = 0; t < mine; t += SUMS) {
    step(t, sums[0]);
    if constexpr (SUMS == 2)
      if (t + 1 < mine) step(t + 1, sums[1]);
  }
  Acc& acc = sums[0];
  if constexpr (SUMS == 2) {
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
      for (int c = 0; c < TN; ++c)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[a][c][v] += sums[1][a][c][v];
  }
  lds_barrier();      // every wave has read its slices: the partial tiles overlap them

  float* const part = reinterpret_cast<float*>(lds);
  {
    float* p = part + wave * (S::PART / 4) + li * S::LDC + 4 * h;
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
      for (int c = 0; c < TN; ++c)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          *reinterpret_cast<float4*>(p + a * 32 * S::LDC + c * 32 + 8 * q) =
              make_float4(acc[a][c][4 * q], acc[a][c][4 * q + 1], acc[a][c][4 * q + 2], acc[a][c][4 * q + 3]);
  }
  lds_barrier();
#pragma unroll
  for (int e = 0; e < (BM * BN / 8 + 64 * WAVES - 1) / (64 * WAVES); ++e) {
    const int idx = e * 64 * WAVES + tid;
    if (BM * BN / 8 % (64 * WAVES) != 0 && idx >= BM * BN / 8) break;
    const int row = idx / (BN / 8), col = idx % (BN / 8) * 8;
    float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
      const float* p = part + w * (S::PART / 4) + row * S::LDC + col;
      const float4 lo = *reinterpret_cast<const float4*>(p), hi = *reinterpret_cast<const float4*>(p + 4);
      v[0] += lo.x; v[1] += lo.y; v[2] += lo.z; v[3] += lo.w;
      v[4] += hi.x; v[5] += hi.y; v[6] += hi.z; v[7] += hi.w;
    }
    epi(0, split, i0 + row, j0 + col, v);
  }
}

template <class T, int BM, int BN, int WAVES, int NS, bool A_K, class Epi>
void launch_slices(SliceArgs g, Epi epi, i64 N, int splits, hipStream_t st) {
  using S = SliceShape<T, BM, BN, WAVES, NS>;
  auto kern = slice_kernel<T, BM, BN, WAVES, NS, A_K, Epi>;
  static const bool configured = lds_limit((const void*)kern, S::LDS);
  (void)configured;
  g.tiles_m = ceil_div(g.M, BM);
  g.slices_per_split = ceil_div(g.slices, splits);
  hipLaunchKernelGGL(kern, dim3((unsigned)((i64)g.tiles_m * ceil_div(N, BN)), (unsigned)splits), dim3(64 * WAVES), S::LDS, st, g, epi);
}

}  // namespace edge
}  // namespace poetx
