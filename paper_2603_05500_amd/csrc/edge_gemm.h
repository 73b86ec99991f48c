// Matrix-core product for shapes the streaming kernels do not take: any sizes, any row stride, any
// alignment of the element type, bf16 (v_mfma_f32_32x32x16_bf16) and fp32 (v_mfma_f32_32x32x2_f32),
// fp32 accumulation in both.
//
//   C[batch](i, j) = sum_k A[batch](i, k) * B[batch](k, j)
//
// An operand is a row-major matrix in memory whose rows may be gathered through a permutation.  It is
// "K major" when the contraction index runs along its rows (contiguous) and "X major" when the output
// index does.  Tiles are loaded through registers, 16 bytes per lane whatever the alignment (element
// aligned vectors: one global load either way), masked at the edges with zeros on both operands so that
// nothing outside the valid ranges takes part, and pass through a two-stage LDS ring with one barrier
// per stage; the loads of the next stage are in flight under the products of this one.
//
// What bounds it: at the sizes it serves the chip is rarely full, so a pass is a chain of latencies (load,
// LDS, matrix product, store).  Hence tile and contraction split follow the problem (dense_plan, apply_tile, grad_plan): 128 x 128, 64 x 64,
// and 32 x 32 with all waves splitting the contraction (each takes its part of every stage; the partial tiles meet in LDS) for the
// smallest, which quarters the chain.
#pragma once
#include "mfma_gemm.h"

namespace poetx {
namespace edge {

using mm::bf16x8;
using mm::floatx16;
using mm::lds_barrier;
using mm::short4v;
using mm::short8v;

// One operand.  Row r of batch bt lies at p + bt * bs + row * ld with row = perm ? perm[bt * rpb + r] : r.
struct Op {
  const void* p;
  i64 ld, bs;
  const int32_t* perm;
  int rows, cols;        // valid extents
  int rows_side;         // != 0: rows (cols) also end at the side of the batch's block
  int cols_side;
  i64 cs;                // strided operands (template flag): distance of neighbouring columns, rows then being ld apart as ever
};

struct Args {
  Op A, B;
  int tiles_m, tiles_n, batches;
  int stages, stages_per_split;   // contraction stages in all and per split
  int rpb, d;                     // rpb > 0: block side of batch bt is min(rpb, d - bt * rpb)
};

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_a2 __attribute__((ext_vector_type(4), aligned(2)));
typedef uint32_t u32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));

__device__ inline u32x4 load16(const uint16_t* p) { return *reinterpret_cast<const u32x4_a2*>(p); }
__device__ inline u32x4 load16(const float* p) { return *reinterpret_cast<const u32x4_a4*>(p); }

// 16 bytes of a row starting at column c >= 0: zeros from column cols on, or altogether if !row_ok.  A branch per lane: lanes that have
// nothing to read read nothing, and whole vectors cost nothing more; a tail is read element by element and waited for.
template <class T>
__device__ __forceinline__ u32x4 load_branched(const T* row, int c, int cols, bool row_ok) {
  constexpr int V = 16 / sizeof(T);
  u32x4 v = {0, 0, 0, 0};
  if (!row_ok || c >= cols) return v;
  if (cols - c >= V) return load16(row + c);   // no sum: the last column may be the last int
  const int n = cols - c;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    if constexpr (sizeof(T) == 4) {
      if (w < n) v[w] = __builtin_bit_cast(uint32_t, row[c + w]);
    } else {
      uint32_t x = 0;
      if (2 * w < n) x = row[c + 2 * w];
      if (2 * w + 1 < n) x |= (uint32_t)row[c + 2 * w + 1] << 16;
      v[w] = x;
    }
  }
  return v;
}

// v without its first n elements, zeros behind them (all zeros from n = 8 on)
__device__ __forceinline__ u32x4 drop_first(const u32x4& v, int n) {
  typedef unsigned long long u64;
  const u64 lo = (u64)v[1] << 32 | v[0], hi = (u64)v[3] << 32 | v[2];
  const int bits = n * 16, in = bits & 63;
  const u64 carry = in ? hi << (64 - in) : 0, l = bits < 64 ? lo >> in | carry : hi >> in, h = bits < 64 ? hi >> in : 0;
  const bool none = bits >= 128;
  u32x4 r;
  r[0] = none ? 0 : (uint32_t)l;
  r[1] = none ? 0 : (uint32_t)(l >> 32);
  r[2] = none ? 0 : (uint32_t)h;
  r[3] = none ? 0 : (uint32_t)(h >> 32);
  return r;
}

// The same load of a bf16 row of at least 8 columns without a branch, in two halves: the load (a vector that would pass the row's end ends there
// instead; a row that is not there is some other one) and, once it is waited for, the mask.
__device__ __forceinline__ u32x4 load_raw(const uint16_t* row, int c, int cols) { return load16(row + (c < cols - 8 ? c : cols - 8)); }
__device__ __forceinline__ u32x4 mask_raw(const u32x4& v, int c, int cols, bool row_ok) {
  const int past = c <= cols - 8 ? 0 : c - (cols - 8);
  return drop_first(v, row_ok && past < 8 ? past : 8);
}

// the same with columns cs elements apart
template <class T>
__device__ inline u32x4 load_strided(const T* row, int c, i64 cs, int cols, bool row_ok) {
  constexpr int V = 16 / sizeof(T);
  u32x4 v = {0, 0, 0, 0};
  if (!row_ok || c >= cols) return v;
#pragma unroll
  for (int e = 0; e < V; ++e) {
    if (e < cols - c) {
      if constexpr (sizeof(T) == 4) v[e] = __builtin_bit_cast(uint32_t, row[(c + e) * cs]);
      else v[e >> 1] |= (uint32_t)row[(c + e) * cs] << (16 * (e & 1));
    }
  }
  return v;
}

// ---- eight consecutive output elements ------------------------------------------------------
__device__ inline void store8(uint16_t* p, const float (&v)[8], int n) {
  const u32x4 o = {mm::pack2_bf16(v[0], v[1]), mm::pack2_bf16(v[2], v[3]), mm::pack2_bf16(v[4], v[5]), mm::pack2_bf16(v[6], v[7])};
  if (n >= 8) {
    *reinterpret_cast<u32x4_a2*>(p) = o;
  } else {
#pragma unroll
    for (int e = 0; e < 7; ++e)
      if (e < n) p[e] = (uint16_t)(o[e >> 1] >> (16 * (e & 1)));
  }
}
__device__ inline void store8(float* p, const float (&v)[8], int n) {
  typedef float f4 __attribute__((ext_vector_type(4), aligned(4)));
  if (n >= 8) {
    *reinterpret_cast<f4*>(p) = f4{v[0], v[1], v[2], v[3]};
    *reinterpret_cast<f4*>(p + 4) = f4{v[4], v[5], v[6], v[7]};
  } else {
#pragma unroll
    for (int e = 0; e < 7; ++e)
      if (e < n) p[e] = v[e];
  }
}

// chunk swizzle of an X-major bf16 tile (see kx_chunk); 32-wide rows need none: the four k rows of a
// transposing read are 64 bytes apart and already fall on different banks
template <int X>
__device__ inline int kx_swz(int c, int k) {
  if constexpr (X >= 64) return mm::kx_chunk<X>(c, k);
  else return c;
}

// Fragment of 32 rows (columns) from x0, k step ks of a 32-deep bf16 sub-tile: K major, or X major through the transposing read
template <int X, bool K_MAJOR>
__device__ __forceinline__ bf16x8 frag_bf16(const char* sub, int x0, int ks) {
  const int lane = threadIdx.x & 63;
  if constexpr (K_MAJOR) {
    const int r = x0 + (lane & 31);
    return *reinterpret_cast<const bf16x8*>(sub + r * 64 + 16 * mm::xk_chunk(2 * ks + (lane >> 5), r));
  } else {
    const int q = lane >> 4, i = lane & 15;
    const int k = 16 * ks + 8 * (q >> 1) + (i >> 2);
    const int c = (x0 >> 3) + 2 * (q & 1) + ((i & 3) >> 1);
    // the swizzle depends on k & 3 only, so the second half (k + 4) uses the same chunk position
    const char* p = sub + k * (X * 2) + 16 * kx_swz<X>(c, k) + 8 * (i & 1);
    const short4v lo = mm::lds_read_tr(p), hi = mm::lds_read_tr(p + 4 * (X * 2));
    const short8v v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8, v);
  }
}

template <class T, int X, int BK>
constexpr int tile_bytes() { return sizeof(T) == 2 ? X * BK * 2 : (X + 4) * BK * 4; }

// WAVES waves: those beyond WGM x WGN split the contraction of a stage
template <class T, int BM, int BN, int BK, int WGM, int WGN, int WAVES>
struct Shape {
  static constexpr int THREADS = 64 * WAVES, WGK = WAVES / (WGM * WGN);
  static constexpr int A_BYTES = tile_bytes<T, BM, BK>(), B_BYTES = tile_bytes<T, BN, BK>();
  static constexpr int STAGE = A_BYTES + B_BYTES;
  static constexpr int LDS = 2 * STAGE;
  static constexpr int TM = BM / WGM / 32, TN = BN / WGN / 32;
  static_assert(WGM * WGN * 32 * (TN * 32 + 4) * 4 <= LDS, "output staging fits the ring");
  static_assert(WGK == 1 || (WGK - 1) * WGM * WGN * TM * TN * 4096 <= LDS, "partial tiles meet in the ring");
};

// How the operands' vectors are loaded; STRIDED and MASKED are about B alone.
// WHOLE: every tile and stage lies inside both operands, nothing is checked.
// MASKED (bf16 rows of at least 8 columns whose count is no multiple of 8; B X major): every stage of the last tile ends in tails, and what is
// branched waits for them -- load_raw, and the mask on the way into LDS.  us, branched / masked: applies of 411 features, b = 256, 28 tokens 6.3 / 5.1;
// 1258, b = 128, 1501 7.2 / 5.9; 524, b = 64, 302 4.9 / 3.9; but 4122, b = 128, 1032 tokens 11.0 / 11.5.
// Elsewhere branches are the better form of an edge, and one stage ahead is enough: the arithmetic of masks and the registers of a second stage cost
// more than they hide (us, masks and two stages / branches and one: fp32 gradients of 2380 features, b = 48, 3925 tokens 57.3 / 46.1; bf16 products of sizes in
// 32s with 1 - 7 tokens 25 % less time, fp32 ones 7 %).  A choice between WHOLE and BRANCHED inside one kernel costs the short launches that are
// not whole up to 5 % (the code), so it is made outside; us, BRANCHED / WHOLE: gradients of 1024 features, b = 64, 512 tokens 4.28 / 3.77; bf16 1024 x 1024 x 512 8.4 / 7.5 and,
// backward, 9.2 / 7.8; fp32 256 x 256 x 512 6.4 / 6.0.
enum Load { BRANCHED, STRIDED, MASKED, WHOLE };

// Epi: __device__ void operator()(int batch, int split, int row, int col, const float (&v)[8]) -- eight
// consecutive columns of one output row, indices inside the batch; it does its own masking.
// bx of total: this workgroup among those of the problem.
template <class T, int BM, int BN, int BK, int WGM, int WGN, int WAVES, bool A_K, bool B_K, class Epi, Load LOAD>
__device__ __forceinline__ void edge_product(const Args& g, const Epi& epi, int bx, int total, int split) {
  using S = Shape<T, BM, BN, BK, WGM, WGN, WAVES>;
  constexpr int V = 16 / sizeof(T), WGK = S::WGK, TM = S::TM, TN = S::TN;
  constexpr bool BF = sizeof(T) == 2;
  constexpr int NTH = S::THREADS, NVA = BM * BK / V / NTH, NVB = BN * BK / V / NTH;
  static_assert(NVA >= 1 && NVB >= 1, "tile too small");
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wk = wave / (WGM * WGN), wm = (wave / WGN) % WGM, wn = wave % WGN;
  const int tiles = g.tiles_m * g.tiles_n;
  // Consecutive workgroups go to the 8 XCDs in turn: give each XCD a contiguous run of tiles (and the tiles of a batch
  // that read the same columns come first), so that shared operand rows meet in one L2.
  const int xcd = bx & 7, per = total >> 3, extra = total & 7;
  const int id = xcd * per + (xcd < extra ? xcd : extra) + (bx >> 3);
  const int batch = id / tiles, tile = id % tiles;
  const int i0 = (tile % g.tiles_m) * BM, j0 = (tile / g.tiles_m) * BN;
  const int side = g.rpb > 0 ? (g.d - batch * g.rpb < g.rpb ? g.d - batch * g.rpb : g.rpb) : 0x7fffffff;

  // ---- loads: vector s of this thread covers row (s * NTH + tid) / VPR of the tile's memory rows
  struct Side {
    const T* base;
    const int32_t* pm;
    i64 ld;
    int rows, cols;
  };
  auto side_of = [&](const Op& o) {
    Side r;
    r.base = (const T*)o.p + (i64)batch * o.bs;
    r.pm = o.perm ? o.perm + (i64)batch * g.rpb : nullptr;
    r.ld = o.ld;
    r.rows = o.rows_side && side < o.rows ? side : o.rows;
    r.cols = o.cols_side && side < o.cols ? side : o.cols;
    return r;
  };
  const Side sa = side_of(g.A), sb = side_of(g.B);
  constexpr int VPRA = (A_K ? BK : BM) / V, VPRB = (B_K ? BK : BN) / V;
  static_assert(LOAD != MASKED || (BF && !B_K), "masked loads are of bf16 rows along the output index");
  u32x4 ra[NVA], rb[NVB];
  // Memory row of this thread's vector (its offset; where there is none, that of the first): fixed for a K-major operand, moving with
  // the stage for an X-major one.
  i64 rowA[NVA], rowB[NVB];
  auto row_at = [&](const Side& s, int r) {
    const int rr = LOAD == WHOLE || r < s.rows ? r : 0;
    return (s.pm ? (i64)s.pm[rr] : (i64)rr) * s.ld;
  };
  auto rowno_a = [&](int s, int kt) { return (A_K ? i0 : kt * BK) + (s * NTH + tid) / VPRA; };
  auto rowno_b = [&](int s, int kt) { return (B_K ? j0 : kt * BK) + (s * NTH + tid) / VPRB; };
  auto col_a = [&](int s, int kt) { return (A_K ? kt * BK : i0) + ((s * NTH + tid) % VPRA) * V; };
  auto col_b = [&](int s, int kt) { return (B_K ? kt * BK : j0) + ((s * NTH + tid) % VPRB) * V; };
  auto rows_at = [&](int kt, bool first) {
    if (!A_K || first) {
#pragma unroll
      for (int s = 0; s < NVA; ++s) rowA[s] = row_at(sa, rowno_a(s, kt));
    }
    if (!B_K || first) {
#pragma unroll
      for (int s = 0; s < NVB; ++s) rowB[s] = row_at(sb, rowno_b(s, kt));
    }
  };
  const int whole_b = tile_inside(j0, BN, sb.cols) ? sb.rows / BK : 0;   // MASKED: stages up to here are whole and need no mask
  auto gload = [&](int kt) {
#pragma unroll
    for (int s = 0; s < NVA; ++s) {
      if constexpr (LOAD == WHOLE) ra[s] = load16(sa.base + rowA[s] + col_a(s, kt));
      else ra[s] = load_branched(sa.base + rowA[s], col_a(s, kt), sa.cols, rowno_a(s, kt) < sa.rows);
    }
#pragma unroll
    for (int s = 0; s < NVB; ++s) {
      if constexpr (LOAD == WHOLE) rb[s] = load16(sb.base + rowB[s] + col_b(s, kt));
      else if constexpr (LOAD == STRIDED) rb[s] = load_strided<T>(sb.base + rowB[s], col_b(s, kt), g.B.cs, sb.cols, rowno_b(s, kt) < sb.rows);
      else if constexpr (LOAD == MASKED) rb[s] = load_raw(sb.base + rowB[s], col_b(s, kt), sb.cols);
      else rb[s] = load_branched(sb.base + rowB[s], col_b(s, kt), sb.cols, rowno_b(s, kt) < sb.rows);
    }
  };
  // ---- LDS layout.  bf16: 32-deep sub-tiles in the swizzled layouts of mfma_gemm.h.  fp32: [k][x], rows of
  // X + 4 floats (the transposing stores of a K-major operand then spread over the banks).
  auto put = [&](char* at, const u32x4& v, int r, int vc, auto X_, bool kmajor) {
    constexpr int X = decltype(X_)::value;
    if constexpr (BF) {
      if (kmajor) *reinterpret_cast<u32x4*>(at + (vc >> 2) * (X * 64) + r * 64 + 16 * mm::xk_chunk(vc & 3, r)) = v;
      else *reinterpret_cast<u32x4*>(at + (r >> 5) * (X * 64) + (r & 31) * (X * 2) + 16 * kx_swz<X>(vc, r & 31)) = v;
    } else {
      float* f = reinterpret_cast<float*>(at);
      if (kmajor) {
#pragma unroll
        for (int e = 0; e < 4; ++e) f[(vc * 4 + e) * (X + 4) + r] = __builtin_bit_cast(float, (uint32_t)v[e]);
      } else {
        *reinterpret_cast<u32x4*>(f + r * (X + 4) + vc * 4) = v;
      }
    }
  };
  auto lstore = [&](int slot, int kt) {
    if constexpr (LOAD == MASKED) {
      if (kt >= whole_b) {
#pragma unroll
        for (int s = 0; s < NVB; ++s) rb[s] = mask_raw(rb[s], col_b(s, kt), sb.cols, rowno_b(s, kt) < sb.rows);
      }
    }
    char* stage = lds + slot * S::STAGE;
#pragma unroll
    for (int s = 0; s < NVA; ++s)
      put(stage, ra[s], (s * NTH + tid) / VPRA, (s * NTH + tid) % VPRA, std::integral_constant<int, BM>{}, A_K);
#pragma unroll
    for (int s = 0; s < NVB; ++s)
      put(stage + S::A_BYTES, rb[s], (s * NTH + tid) / VPRB, (s * NTH + tid) % VPRB, std::integral_constant<int, BN>{}, B_K);
  };

  floatx16 acc[TM][TN];
#pragma unroll
  for (int a = 0; a < TM; ++a)
#pragma unroll
    for (int c = 0; c < TN; ++c)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[a][c][v] = 0.f;

  const int li = lane & 31, h = lane >> 5;
  auto multiply = [&](int slot) {
    const char* sA = lds + slot * S::STAGE;
    const char* sB = sA + S::A_BYTES;
    if constexpr (BF) {
      constexpr int SUBS = BK / 32 / WGK;      // 32-deep sub-tiles per wave
      static_assert(SUBS >= 1, "a wave of a split contraction takes whole sub-tiles");
#pragma unroll
      for (int u = 0; u < SUBS; ++u) {
        const int sub = wk * SUBS + u;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
          bf16x8 fa[TM], fb[TN];
#pragma unroll
          for (int a = 0; a < TM; ++a)
            fa[a] = frag_bf16<BM, A_K>(sA + sub * (BM * 64), wm * (BM / WGM) + a * 32, ks);
#pragma unroll
          for (int c = 0; c < TN; ++c)
            fb[c] = frag_bf16<BN, B_K>(sB + sub * (BN * 64), wn * (BN / WGN) + c * 32, ks);
#pragma unroll
          for (int a = 0; a < TM; ++a)
#pragma unroll
            for (int c = 0; c < TN; ++c)
              acc[a][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[c], fa[a], acc[a][c], 0, 0, 0);
        }
      }
    } else {
      constexpr int KW = BK / WGK;             // depth of a stage that one wave takes
      const float* fA = reinterpret_cast<const float*>(sA) + (wk * KW + h) * (BM + 4) + wm * (BM / WGM) + li;
      const float* fB = reinterpret_cast<const float*>(sB) + (wk * KW + h) * (BN + 4) + wn * (BN / WGN) + li;
#pragma unroll
      for (int kk = 0; kk < KW; kk += 2) {
        float fa[TM], fb[TN];
#pragma unroll
        for (int a = 0; a < TM; ++a) fa[a] = fA[kk * (BM + 4) + a * 32];
#pragma unroll
        for (int c = 0; c < TN; ++c) fb[c] = fB[kk * (BN + 4) + c * 32];
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
          for (int c = 0; c < TN; ++c)
            acc[a][c] = __builtin_amdgcn_mfma_f32_32x32x2f32(fb[c], fa[a], acc[a][c], 0, 0, 0);
      }
    }
  };

  const int k0 = split * g.stages_per_split;
  const int k1 = k0 + g.stages_per_split < g.stages ? k0 + g.stages_per_split : g.stages;
  if (k0 < k1) {
    // stage kt + 1 is requested while kt is multiplied: its registers were written to LDS a stage ago
    rows_at(k0, true);
    gload(k0);
    if (k0 + 1 < k1) rows_at(k0 + 1, false);
    lstore(0, k0);
    lds_barrier();
    for (int kt = k0; kt < k1; ++kt) {
      const int slot = (kt - k0) & 1;
      if (kt + 1 < k1) {
        gload(kt + 1);
        if (kt + 2 < k1) rows_at(kt + 2, false);
      }
      multiply(slot);
      if (kt + 1 < k1) lstore(slot ^ 1, kt + 1);   // read last before the previous barrier
      lds_barrier();
    }
  }

  if constexpr (WGK > 1) {
    // the partial tiles of the waves that share an output piece meet in LDS; wave 0 adds them in order
    constexpr int TILE_F = TM * TN * 1024;
    float* part = reinterpret_cast<float*>(lds);
    const int piece = wm * WGN + wn;
    if (wk > 0) {
      float* dst = part + ((wk - 1) * WGM * WGN + piece) * TILE_F + lane * 4;
#pragma unroll
      for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int c = 0; c < TN; ++c)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            *reinterpret_cast<float4*>(dst + ((a * TN + c) * 4 + q) * 256) =
                make_float4(acc[a][c][4 * q], acc[a][c][4 * q + 1], acc[a][c][4 * q + 2], acc[a][c][4 * q + 3]);
    }
    lds_barrier();
    if (wk == 0) {
#pragma unroll
      for (int w = 0; w < WGK - 1; ++w) {
        const float* src = part + (w * WGM * WGN + piece) * TILE_F + lane * 4;
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
          for (int c = 0; c < TN; ++c)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const float4 p = *reinterpret_cast<const float4*>(src + ((a * TN + c) * 4 + q) * 256);
              acc[a][c][4 * q] += p.x;
              acc[a][c][4 * q + 1] += p.y;
              acc[a][c][4 * q + 2] += p.z;
              acc[a][c][4 * q + 3] += p.w;
            }
      }
    }
    // the areas below overlap the partial tiles of other pieces: every wave has read its own
    if (WGM * WGN > 1) lds_barrier();
    else asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if (wk > 0) return;
  }

  // A lane holds one output row and four columns per register group: written like that, an instruction would touch
  // 32 rows with 32 bytes each.  The wave passes 32 rows at a time through an LDS area of its own (fp32) and reads
  // them back row by row, so that neighbouring lanes hold neighbouring pieces of a row -- eight columns each -- for the
  // epilogue's loads and stores (8192 x 4090 apply at b = 256: 105 -> 94 us).
  constexpr int CW = TN * 32, LDC = CW + 4, LPR = CW / 8, RPP = 64 / LPR;
  float* stg = reinterpret_cast<float*>(lds) + wave * (32 * LDC);
#pragma unroll
  for (int a = 0; a < TM; ++a) {
#pragma unroll
    for (int c = 0; c < TN; ++c)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<float4*>(stg + li * LDC + c * 32 + 8 * q + 4 * h) =
            make_float4(acc[a][c][4 * q], acc[a][c][4 * q + 1], acc[a][c][4 * q + 2], acc[a][c][4 * q + 3]);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the wave's own writes
#pragma unroll
    for (int r0 = 0; r0 < 32; r0 += RPP) {
      const int r = r0 + lane / LPR, c8 = (lane % LPR) * 8;
      const float4 lo = *reinterpret_cast<const float4*>(stg + r * LDC + c8), hi = *reinterpret_cast<const float4*>(stg + r * LDC + c8 + 4);
      const float v[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
      epi(batch, split, i0 + wm * (BM / WGM) + a * 32 + r, j0 + wn * (BN / WGN) + c8, v);
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // read back before the area is rewritten
  }
}

template <class T, int BM, int BN, int BK, int WGM, int WGN, int WAVES, bool A_K, bool B_K, class Epi, Load LOAD>
__global__ __launch_bounds__((Shape<T, BM, BN, BK, WGM, WGN, WAVES>::THREADS)) void edge_kernel(Args g, Epi epi, int total, int first) {
  edge_product<T, BM, BN, BK, WGM, WGN, WAVES, A_K, B_K, Epi, LOAD>(g, epi, first + (int)blockIdx.x, total, blockIdx.y);
}

// Two problems of one shape in one launch: the first n0 workgroups of a row of the grid take g0, the rest g1.
template <class T, int BM, int BN, int BK, int WGM, int WGN, int WAVES, bool A_K, bool B_K, class Epi, Load LOAD>
__global__ __launch_bounds__((Shape<T, BM, BN, BK, WGM, WGN, WAVES>::THREADS)) void edge_pair_kernel(Args g0, Args g1, Epi e0, Epi e1, int n0, int total, int first) {
  const int bx = first + (int)blockIdx.x;
  const bool second = bx >= n0;
  const Args g = second ? g1 : g0;
  const Epi epi = second ? e1 : e0;
  const int split = blockIdx.y;
  if (split * g.stages_per_split >= g.stages) return;
  edge_product<T, BM, BN, BK, WGM, WGN, WAVES, A_K, B_K, Epi, LOAD>(g, epi, second ? bx - n0 : bx, second ? total - n0 : n0, split);
}

// An apply and two problems of one shape (the block gradients of both sides) in one launch: what a small layer's backward has left once dA is there.  Each is a chain of
// latencies that leaves most of the chip idle, and they do not depend on each other.  Workgroups: n0 of g0 for each of its splits, n1 of g1, then those of the apply.
template <class T, int ABM, int ABK, int AWG, int AWAVES, Load ALOAD, class AEpi, int BK, Load LOAD, class Epi>
__global__ __launch_bounds__(256) void edge_apply_pair_kernel(Args ga, AEpi ea, Args g0, Args g1, Epi e0, Epi e1, int n0, int n1, int pairs0, int pairs, int na) {
  int bx = blockIdx.x;
  if (bx < pairs) {
    const bool second = bx >= pairs0;
    const Args g = second ? g1 : g0;
    const Epi epi = second ? e1 : e0;
    if (second) bx -= pairs0;
    const int n = second ? n1 : n0, split = bx / n;
    edge_product<T, 32, 32, BK, 1, 1, 4, true, true, Epi, LOAD>(g, epi, bx - split * n, n, split);
  } else {
    if (threadIdx.x >= 64 * AWAVES) return;
    edge_product<T, ABM, ABM, ABK, AWG, AWG, AWAVES, true, false, AEpi, ALOAD>(ga, ea, bx - pairs, na, 0);
  }
}

// ---- host side -------------------------------------------------------------------------------
enum Tile { TILE_32 = 0, TILE_64 = 1, TILE_128 = 2, TILE_64D = 3 };   // 64D: 64 x 64, deeper stages, sixteen waves (fp32 dense products)

struct Plan {
  Tile tile;
  int splits;
};

constexpr int kCUs = 256;

inline i64 tile_count(i64 batches, i64 M, i64 N, int t) { return batches * ((M + t - 1) / t) * ((N + t - 1) / t); }
// contraction depth of a stage; fp32 halves it, which keeps as many workgroups per CU as in bf16
constexpr int stage_depth(Tile t, size_t es) { return (t == TILE_32 || t == TILE_64D ? 128 : 64) * 2 / (int)es; }

struct Problem {
  i64 batches, M, N, K;
};
inline bool lds_limit(const void* kern, int bytes) { return hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, bytes) == hipSuccess; }
inline void tile_args(Args& g, const Problem& q, int BM, int BN, int BK, int splits) {
  g.tiles_m = ceil_div(q.M, BM);
  g.tiles_n = ceil_div(q.N, BN);
  g.batches = (int)q.batches;
  g.stages = ceil_div(q.K, BK);
  g.stages_per_split = ceil_div(g.stages, splits);
}

// WHOLE: do all tiles and stages lie inside the operands?
template <int BM, int BN, int BK, bool A_K, bool B_K>
bool whole_tiles(const Args& g) {
  const i64 M = (i64)g.tiles_m * BM, N = (i64)g.tiles_n * BN, K = (i64)g.stages * BK;
  return (g.rpb == 0 || g.d % g.rpb == 0) && M <= (A_K ? g.A.rows : g.A.cols) && K <= (A_K ? g.A.cols : g.A.rows) &&
         N <= (B_K ? g.B.rows : g.B.cols) && K <= (B_K ? g.B.cols : g.B.rows);
}

template <class T, int BM, int BN, int BK, int WGM, int WGN, int WAVES, bool A_K, bool B_K, Load LOAD = BRANCHED, class Epi>
void launch_shape(Args g, Epi epi, i64 batches, i64 M, i64 N, i64 K, int splits, hipStream_t st) {
  using S = Shape<T, BM, BN, BK, WGM, WGN, WAVES>;
  tile_args(g, Problem{batches, M, N, K}, BM, BN, BK, splits);
  const i64 total = batches * g.tiles_m * g.tiles_n;
  auto go = [&](auto kern) {
    launch_in_rows(total, [&](int first, unsigned count) {
      hipLaunchKernelGGL(kern, dim3(count, (unsigned)splits), dim3(S::THREADS), S::LDS, st, g, epi, (int)total, first);
    });
  };
  if constexpr (LOAD == BRANCHED) {
    if (whole_tiles<BM, BN, BK, A_K, B_K>(g)) {
      auto kern = edge_kernel<T, BM, BN, BK, WGM, WGN, WAVES, A_K, B_K, Epi, WHOLE>;
      static const bool configured = lds_limit((const void*)kern, S::LDS);
      (void)configured;
      return go(kern);
    }
  }
  auto kern = edge_kernel<T, BM, BN, BK, WGM, WGN, WAVES, A_K, B_K, Epi, LOAD>;
  static const bool configured = lds_limit((const void*)kern, S::LDS);
  (void)configured;
  go(kern);
}

template <class T, int BM, int BN, int BK, int WGM, int WGN, int WAVES, bool A_K, bool B_K, class Epi>
void launch_pair_shape(Args g0, Args g1, Epi e0, Epi e1, const Problem& q0, const Problem& q1, int s0, int s1, hipStream_t st) {
  using S = Shape<T, BM, BN, BK, WGM, WGN, WAVES>;
  tile_args(g0, q0, BM, BN, BK, s0);
  tile_args(g1, q1, BM, BN, BK, s1);
  const i64 n0 = q0.batches * g0.tiles_m * g0.tiles_n, n1 = q1.batches * g1.tiles_m * g1.tiles_n;
  const bool whole0 = whole_tiles<BM, BN, BK, A_K, B_K>(g0), whole1 = whole_tiles<BM, BN, BK, A_K, B_K>(g1);
  // Only one of them whole and the chip full of either, on the largest tile: each on its own kernel (gradients of 8192 and 3072 features, 4090 tokens, the latter's padded: 74 us together, 46 + 20 so).
  // Not otherwise, the second launch costs more: halves of the backward, together / apart, 144 and 3136 features, b = 32, 1792 tokens 11.5 / 15.3 us; over 300 of them on smaller tiles 4 % more apart, on the
  // largest with a side of 128 to 256 workgroups 1.3 % more, with more on both sides 1 % less (14 % at best).
  if (BM == 128 && whole0 != whole1 && n0 * s0 > kCUs && n1 * s1 > kCUs) {
    launch_shape<T, BM, BN, BK, WGM, WGN, WAVES, A_K, B_K>(g0, e0, q0.batches, q0.M, q0.N, q0.K, s0, st);
    launch_shape<T, BM, BN, BK, WGM, WGN, WAVES, A_K, B_K>(g1, e1, q1.batches, q1.M, q1.N, q1.K, s1, st);
    return;
  }
  auto go = [&](auto kern) {
    launch_in_rows(n0 + n1, [&](int first, unsigned count) {
      hipLaunchKernelGGL(kern, dim3(count, (unsigned)(s0 > s1 ? s0 : s1)), dim3(S::THREADS), S::LDS, st, g0, g1, e0, e1, (int)n0, (int)(n0 + n1), first);
    });
  };
  // once per kernel instance; a function-local static is initialised exactly once, whichever thread gets there first
  if (whole0 && whole1) {
    auto kern = edge_pair_kernel<T, BM, BN, BK, WGM, WGN, WAVES, A_K, B_K, Epi, WHOLE>;
    static const bool configured = lds_limit((const void*)kern, S::LDS);
    (void)configured;
    go(kern);
  } else {
    auto kern = edge_pair_kernel<T, BM, BN, BK, WGM, WGN, WAVES, A_K, B_K, Epi, BRANCHED>;
    static const bool configured = lds_limit((const void*)kern, S::LDS);
    (void)configured;
    go(kern);
  }
}

// Applies on the smallest tile: the contraction is a block, and a stage no deeper than it (masked halves of a stage cost a launch
// some 0.4 us).  Strided bf16 loads are eight accesses each: four waves share those of 64 features, whose shallow stage has two (1280 features,
// b = 64, 86 tokens 8.4 / 7.6 us; b = 32 the other way).
template <class T, bool A_K, bool B_K, Load LOAD, class Epi>
void launch_apply_32(const Args& g, Epi epi, i64 batches, i64 M, i64 N, i64 K, hipStream_t st) {
  constexpr int D = 128 / (int)sizeof(T);
  if (K > D || (sizeof(T) == 2 && LOAD == STRIDED && 2 * K > D)) launch_shape<T, 32, 32, 2 * D, 1, 1, 4, A_K, B_K, LOAD>(g, epi, batches, M, N, K, 1, st);
  else if constexpr (sizeof(T) == 4) launch_shape<T, 32, 32, D, 1, 1, 4, A_K, B_K, LOAD>(g, epi, batches, M, N, K, 1, st);
  else launch_shape<T, 32, 32, D, 1, 1, 2, A_K, B_K, LOAD>(g, epi, batches, M, N, K, 1, st);
}
template <class T, bool A_K, bool B_K, Load LOAD, class Epi>
void launch_apply(const Args& g, Epi epi, i64 batches, i64 M, i64 N, i64 K, Tile t, hipStream_t st) {
  constexpr int D = 128 / (int)sizeof(T);
  if (t == TILE_128) launch_shape<T, 128, 128, D, 2, 2, 4, A_K, B_K, LOAD>(g, epi, batches, M, N, K, 1, st);
  else if (t == TILE_64) launch_shape<T, 64, 64, D, 2, 2, 4, A_K, B_K, LOAD>(g, epi, batches, M, N, K, 1, st);
  else launch_apply_32<T, A_K, B_K, LOAD>(g, epi, batches, M, N, K, st);
}

// Dense products (long contractions) have twice the waves on their larger tiles, halves of which split every stage: what
// bounds the plain ones are the latencies of one or two waves per SIMD (fp32 1024 x 1024 x 2048, 64 x 64: 53.0 -> 49.2 us; bf16 1024 x 1536 x 3001,
// 128 x 128: 44 -> 33; block gradients on 128 x 128 lose: 69 -> 95).  Not so 128 x 128 of bf16 with A K major (B = W A): 8192-deep products of 4192 x 1567
// 291 / 199 us with eight waves / four, 7488 x 1984 x 3821 275 / 207; with A X major 7936 x 7872 x 734 169 / 190, 6560 x 3712 x 881 88 / 101.
enum Use { DENSE, GRAD };
template <class T, bool A_K, bool B_K, Use USE, class Epi>
void launch(const Args& g, Epi epi, i64 batches, i64 M, i64 N, i64 K, Plan p, hipStream_t st) {
  constexpr int D = 128 / (int)sizeof(T), W = USE == DENSE ? 8 : 4;   // D: stage_depth
  if constexpr (USE == DENSE && sizeof(T) == 4) {
    if (p.tile == TILE_64D) return launch_shape<T, 64, 64, 2 * D, 2, 2, 16, A_K, B_K>(g, epi, batches, M, N, K, p.splits, st);
  }
  if (p.tile == TILE_128) launch_shape<T, 128, 128, D, 2, 2, sizeof(T) == 2 && A_K ? 4 : W, A_K, B_K>(g, epi, batches, M, N, K, p.splits, st);
  else if (p.tile == TILE_64) launch_shape<T, 64, 64, D, 2, 2, W, A_K, B_K>(g, epi, batches, M, N, K, p.splits, st);
  else launch_shape<T, 32, 32, 2 * D, 1, 1, sizeof(T) == 4 ? W : 4, A_K, B_K>(g, epi, batches, M, N, K, p.splits, st);
}

// two problems planned onto the same tile
template <class T, bool A_K, bool B_K, class Epi>
void launch_pair(const Args& g0, const Args& g1, Epi e0, Epi e1, const Problem& q0, const Problem& q1, Plan p0, Plan p1, hipStream_t st) {
  constexpr int D = 128 / (int)sizeof(T);
  if (p0.tile == TILE_128) launch_pair_shape<T, 128, 128, D, 2, 2, 4, A_K, B_K>(g0, g1, e0, e1, q0, q1, p0.splits, p1.splits, st);
  else if (p0.tile == TILE_64) launch_pair_shape<T, 64, 64, D, 2, 2, 4, A_K, B_K>(g0, g1, e0, e1, q0, q1, p0.splits, p1.splits, st);
  else launch_pair_shape<T, 32, 32, 2 * D, 1, 1, 4, A_K, B_K>(g0, g1, e0, e1, q0, q1, p0.splits, p1.splits, st);
}

// the apply qa (ABM x ABM tiles) beside two gradients on 32 x 32 tiles
template <class T, int ABM, int ABK, int AWG, int AWAVES, bool MASKS, class AEpi, class Epi>
void launch_apply_pair(Args ga, AEpi ea, const Problem& qa, Args g0, Args g1, Epi e0, Epi e1, const Problem& q0, const Problem& q1, int s0, int s1, hipStream_t st) {
  constexpr int BK = 256 / (int)sizeof(T);
  using S = Shape<T, 32, 32, BK, 1, 1, 4>;
  using SA = Shape<T, ABM, ABM, ABK, AWG, AWG, AWAVES>;
  constexpr int LDS = S::LDS > SA::LDS ? S::LDS : SA::LDS;
  tile_args(ga, qa, ABM, ABM, ABK, 1);
  tile_args(g0, q0, 32, 32, BK, s0);
  tile_args(g1, q1, 32, 32, BK, s1);
  const int na = (int)qa.batches * ga.tiles_m * ga.tiles_n, n0 = (int)q0.batches * g0.tiles_m * g0.tiles_n, n1 = (int)q1.batches * g1.tiles_m * g1.tiles_n;
  // no split without stages
  s0 = ceil_div(g0.stages, g0.stages_per_split);
  s1 = ceil_div(g1.stages, g1.stages_per_split);
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3((unsigned)(n0 * s0 + n1 * s1 + na)), dim3(256), LDS, st, ga, ea, g0, g1, e0, e1, n0, n1, n0 * s0, n0 * s0 + n1 * s1, na);
  };
  if constexpr (!MASKS) {
    if (whole_tiles<ABM, ABM, ABK, true, false>(ga) && whole_tiles<32, 32, BK, true, true>(g0) && whole_tiles<32, 32, BK, true, true>(g1)) {
      auto kern = edge_apply_pair_kernel<T, ABM, ABK, AWG, AWAVES, WHOLE, AEpi, BK, WHOLE, Epi>;
      static const bool configured = lds_limit((const void*)kern, LDS);
      (void)configured;
      return go(kern);
    }
  }
  auto kern = edge_apply_pair_kernel<T, ABM, ABK, AWG, AWAVES, MASKS ? MASKED : BRANCHED, AEpi, BK, BRANCHED, Epi>;
  static const bool configured = lds_limit((const void*)kern, LDS);
  (void)configured;
  go(kern);
}

}  // namespace edge
}  // namespace poetx
