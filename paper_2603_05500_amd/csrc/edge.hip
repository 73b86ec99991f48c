// The dense product, the structured apply and the block gradient for every shape the streaming kernels do
// not take (small blocks, ragged tails, token counts and alignments of any kind, fp32 tensors), on the
// edge-handling matrix-core product of edge_gemm.h.  The plain fp32-FMA kernels they replace here used
// 64 x 64 x 16 tiles with one scalar load per element and one workgroup per output tile whatever the
// contraction: 44 TFLOP/s at 2048 x 5632 x 1999 bf16, and 149 us for the 22 block gradients of 1376 features
// over 1024 tokens.
#include "edge_slices.h"

namespace poetx {
namespace {

using namespace edge;

inline i64 min64(i64 a, i64 b) { return a < b ? a : b; }

// ---- plans -------------------------------------------------------------------------------------
// Tile of an apply (a contraction as short as a block): the largest one that still gives three quarters of the CUs a workgroup -- a larger tile
// halves the operand traffic, an idle CU costs more than that.
Tile apply_tile(i64 batches, i64 M, i64 N) {
  if (M > 64 && N > 64 && tile_count(batches, M, N, 128) >= kCUs * 3 / 4) return TILE_128;
  if (M > 32 && N > 32 && tile_count(batches, M, N, 64) >= kCUs * 3 / 4) return TILE_64;
  return TILE_32;
}

// Dense products on the sliced kernel (edge_slices.h): tile and contraction split priced together.  A workgroup's wave takes `lone` us for a slice when the
// workgroup has a CU to itself (`cold` more where the weight is larger than the L2s would keep) and `shared` for each of the workgroups of
// the fullest CU, each of which adds `tail`, on top of `base` for the launch, the first loads and the last stores.  A split adds a launch of `reduce` us with its gap and the
// fp32 parts, written and read; it keeps more slices than a workgroup has waves, and no more than four workgroups per CU (parts of 16 MB at most).  Products of large fp32 weights take no
// less than their operands' way from the L2s, 10 TB/s: without that the smallest tile was priced at half of its time (13312 x 712, 14016 deep 4.5 ms, on 64 x 64 tiles 2.3; 3913 such products: 5.5 % slower than the best tile on average, now 1.2).
// The constants are fitted to 1750 products of 128 - 14336 rows, 1 - 4096 columns and contractions of 128 - 14336, both directions, each timed with every tile and up to sixteen
// splits on operands in the caches but for the large weights: the choice is 1.3 % slower than the best one on average, and takes a third less time than the edge kernel under its own plan (fp32 33 %,
// bf16 36 %).  Whole steps gain as much with 700 MB of operands in turn (1376 x 512, 1024 tokens 71.5 / 58.0 us, on the same operands 67.0 / 55.3; fp32 1024 x 768, 1001 112 / 86, 106 / 82).
// us, edge kernel / here: fp32 1024 x 768 x 1001 29.0 / 18.0 and, backward, 29.7 (with its reduce) / 21; 256 x 256 x 512 6.0 / 4.3; bf16 1376 x 512 x 1024 9.1 / 6.4 and 11.2 / 5.6;
// 768 x 1024 x 500 9.0 / 5.1; 1536 x 1536 x 3000 40.3 / 37.7.
struct SliceCost {
  int bm, bn, waves_log2;
  double base, lone, shared, tail, cold, reduce, parts;
};
enum SliceTile { SLICES_32 = 0, SLICES_32x64 = 1, SLICES_64 = 2, SLICES_64x32 = 3, EDGE_TILES = -1 };
constexpr SliceCost kSlicesF32[] = {{32, 32, 3, 2.5, 0.16, 0.50, 0.83, 0.26, 2.7, 1.0e-6}, {32, 64, 2, 3.4, 0.41, 0.535, 0.45, 0.22, 2.7, 1.0e-6}, {64, 64, 2, 4.0, 0.975, 0.975, 0.25, 0.07, 2.7, 2.0e-6}};
constexpr SliceCost kSlicesBf16[] = {{32, 32, 3, 1.73, 0.01, 0.52, 0.51, 0.35, 3.2, 0.8e-6}, {32, 64, 2, 2.05, 0.03, 0.345, 0.45, 0.11, 3.2, 0.8e-6}, {64, 64, 2, 1.8, 0.43, 0.445, 1.17, 0.09, 3.2, 1.0e-6}};
// Up to 32 columns of a large bf16 weight are bound by the reads of it.  Where its rows are the contraction (dA = W^T dB) 32 of them are half a cache line, so 64 go to
// a workgroup: 7168 x 12800, one token 37.4 us, on 32 x 32 64.4; 9728 x 4096, 5: 21.0 / 26.2.  Fitted to 230 products like the above, 3 % slower than the best on average.
constexpr SliceCost kSlicesFew[] = {{32, 32, 3, 1.50, 0.67, 0.68, 0.53, 0, 3.3, 1.8e-6}, {64, 32, 2, 1.20, 0.04, 0.59, 0.57, 0, 4.75, 1.3e-6}};
struct SlicePlan {
  SliceTile tile;
  int splits;
};
constexpr double kLargeWeight = 6.3e6;         // bytes
// sizes the kernel takes (operands on 16-byte boundaries besides, which the caller looks at): whole slices, rows in whole 16-byte vectors
bool slices_take(int dtype, i64 M, i64 ld_w, i64 act_cols, i64 K) {
  const i64 es = dtype == POETX_F32 ? 4 : 2;
  return K * es % 64 == 0 && ld_w * es % 16 == 0 && act_cols % 8 == 0 && ld_w < (1 << 22) && act_cols < (1 << 22) && tile_count(1, M, act_cols, 32) < (1 << 21);
}
struct EdgePrice {
  double us;
  Plan plan;
};
EdgePrice edge_price(int dtype, i64 M, i64 N, i64 K);
// ceil(x / s) for s up to 16 and x < 2^31 without a division: every linear call prices its products.  The half keeps the product's rounding off whole numbers.
constexpr double kInverse[] = {0,       1.0 / 1, 1.0 / 2,  1.0 / 3,  1.0 / 4,  1.0 / 5,  1.0 / 6,  1.0 / 7, 1.0 / 8,
                               1.0 / 9, 1.0 / 10, 1.0 / 11, 1.0 / 12, 1.0 / 13, 1.0 / 14, 1.0 / 15, 1.0 / 16};
inline unsigned share(unsigned x, unsigned s) { return (unsigned)(((double)(x + s) - 0.5) * kInverse[s]); }
// edge: the edge kernel's price of the same product, from a caller that has it
SlicePlan slice_plan(int dtype, int trans_w, i64 M, i64 N, i64 K, const EdgePrice* edge = nullptr) {
  const bool f = dtype == POETX_F32;
  const int es = f ? 4 : 2;
  const unsigned slices = (unsigned)slice_count((int)K, es);
  const bool large = (double)M * (double)K * (double)es > kLargeWeight;
  SlicePlan best{SLICES_32, 1};
  double least = 0;
  auto price = [&](const SliceCost& c, SliceTile tile) {
    const unsigned count = (unsigned)(((M + c.bm - 1) / c.bm) * ((N + c.bn - 1) / c.bn));     // below 2^21, see slices_take
    const double lone = c.lone + (large ? c.cold : 0), traffic = (c.bm + c.bn) * 4e-7 * (double)K;
    for (unsigned s = 1; s <= 16; ++s) {
      const unsigned each = share(slices, s);
      if (s > 1 && (each <= 1u << c.waves_log2 || count * s > 4 * kCUs)) break;
      const unsigned splits = (slices + each - 1) / each;      // no empty split
      const double per_cu = (double)((count * splits + kCUs - 1) / kCUs), stage = per_cu * c.shared;
      double us = c.base + (double)((each + (1u << c.waves_log2) - 1) >> c.waves_log2) * (lone > stage ? lone : stage) + c.tail * per_cu;
      if (f && large && us < (double)count * traffic) us = (double)count * traffic;
      if (splits > 1) us += c.reduce + c.parts * (double)splits * (double)M * (double)N;
      if (least == 0 || us < least) { least = us; best = SlicePlan{tile, (int)splits}; }
    }
  };
  if (!f && large && N <= 32) {
    price(kSlicesFew[trans_w ? 1 : 0], trans_w ? SLICES_64x32 : SLICES_32);
    return best;
  }
  for (int i = 0; i < 3; ++i) {
    const SliceCost& c = f ? kSlicesF32[i] : kSlicesBf16[i];
    if (i == 0 || (2 * M > c.bm && 2 * N > c.bn)) price(c, (SliceTile)i);    // not where half of the tile would be idle
  }
  // The edge kernel's larger tiles where they still are the better ones, by 26000 products of 64 - 16384 rows and contractions and 1 - 16384 columns timed on both:
  // - Many tiles of a short contraction are bound by their output, and a workgroup here keeps its stores for the end.  fp32 (us, edge / here): 5632 x 10328, 96 deep 140 / 188; 11648 x 3384, 96 107 / 133; bf16
  //   11456 x 12424, 64 96 / 190; 2816 x 10840, 96 34 / 43; 8640 x 1208, 224 26.7 / 28.0.  fp32 up to 160 of depth and two 64 x 64 tiles per CU, bf16 from 384 tiles of 128 x 128 priced 30 % below: of those
  //   products 0.12 and 0.17 % slower than the better kernel on average (0.6 and 1.3 % without these rules; at most 26 %, not 100 %).
  // - Large bf16 weights: 128 x 128 tiles read each operand half as often.  They stay unless this price is a quarter below theirs.
  // - bf16 on 150 to 384 tiles of 128 x 128 (4000 products of 32 - 384 of depth, 128 - 9600 rows and 200 - 16000 columns, whole calls of each; us, edge / here): up to 64 of depth forward 1792 x 2560 10.1 / 11.4,
  //   300 tiles and more 1.3 to 1.9 dearer here, backward 0.4 up to one tile per CU and cheaper beyond.  Deeper ones only forward, where the price is 60 % below: 128 deep on 340 tiles and more 0.8 dearer here; backward up to 3 cheaper.
  //   Slower than the better kernel on average: 1.9 -> 0.23 % forward, 0.33 -> 0.14 % backward.
  if (f) {
    if (K <= 160 && tile_count(1, M, N, 64) >= 2 * kCUs) best.tile = EDGE_TILES;
    return best;
  }
  const i64 tiles = tile_count(1, M, N, 128);
  const bool middle = !large && tiles >= 150 && tiles < 384 && M >= 128 && N >= 200;
  if (middle && K <= 64) {
    if (!trans_w || tiles <= kCUs) best.tile = EDGE_TILES;
  } else if (large || tiles >= 384 || (middle && !trans_w && K <= 256)) {
    const EdgePrice e = edge ? *edge : edge_price(dtype, M, N, K);
    if (e.plan.tile == TILE_128 && e.us < (large ? 1.25 : middle ? 0.4 : 0.7) * least) best.tile = EDGE_TILES;
  }
  return best;
}

// Dense products of the edge kernel: tile and contraction split priced together.  A workgroup takes `lone` us for a stage when it has a CU to itself (`cold` more
// where the weight is larger than the L2s would keep) and `shared` for each of the workgroups on its CU, of which the fullest CU counts; `fill` stages
// more to fill the ring and to store.  A split adds a launch of `reduce` us with its gap and its fp32 parts, written and read at 4 TB/s.
// The constants are fitted to 1520 products of 128 - 14336 rows, 1 - 5000 columns and contractions of 128 - 14336, both directions, weights over 6 MB read from
// memory, each timed with every tile and split: the choice is 1 % slower than the best one on average and takes 10 % (fp32) and 25 % (bf16) less time than a rule
// that takes the largest tile to fill three quarters of the CUs, with four waves each, and then the split.  us of launches one after the other on the same operands (inside a
// step they come from further away: the first is 30.2 there), tile / splits (64D: 64 x 64 with sixteen waves), before the slices above took these sizes, all but the last; operands off 16-byte
// boundaries and contractions of no whole slices still run so:
// fp32 1024 x 768 x 1001 64D/1 27.4, 64/3 29.8, 32/1 31.2; 256 x 256 x 512 32/1 6.2, 32/2 7.4; bf16 1376 x 512 x 1024 64/1 9.6, 32/1 10.7, 128/1 13.8;
// 1024 x 1536 x 3001 64/1 24.7, 128/2 34.6; 4096 x 14336 x 64 64/12 34.0, 64/8 37.3; 4192 x 8000 x 1567 128/1 200, 128/4 228, 64/1 275.
// Up to 32 columns of a large weight are bound by its reads, for which this price is too coarse (up to 12 % slower than four workgroups per CU): as many splits as
// give each CU four workgroups of at least four stages (5632 x 8192 x 24 32/5 25.8, 32/4 29.7; fp32 6208 x 3072 x 2 32/5 27.6, 32/3 33.2).
struct TileCost {
  Tile tile;
  int side;
  double lone, shared;
};
EdgePrice edge_price(int dtype, i64 M, i64 N, i64 K) {
  static const TileCost f32[] = {{TILE_32, 32, 0.70, 0.51}, {TILE_64, 64, 1.51, 0.66}, {TILE_64D, 64, 1.57, 1.46}, {TILE_128, 128, 2.69, 2.32}};
  static const TileCost bf16[] = {{TILE_32, 32, 0.58, 0.31}, {TILE_64, 64, 0.58, 0.35}, {TILE_128, 128, 1.14, 0.62}};
  const bool f = dtype == POETX_F32;
  const size_t es = f ? 4 : 2;
  const double fill = f ? 0.94 : 1.1, reduce = f ? 1.95 : 2.3;
  const bool large = (double)M * (double)K * (double)es > kLargeWeight;
  const double cold = large ? (f ? 0.63 : 0.39) : 0;
  EdgePrice best{0, {TILE_32, 1}};
  for (int t = 0; t < (f ? 4 : 3); ++t) {
    const TileCost& c = f ? f32[t] : bf16[t];
    if (c.side > 32 && (2 * M <= c.side || 2 * N <= c.side)) continue;   // half of it idle
    const i64 count = tile_count(1, M, N, c.side);
    const unsigned depth = (unsigned)stage_depth(c.tile, es), stages = ((unsigned)K + depth - 1) / depth;
    const i64 most = (c.tile == TILE_128 ? 2 : 4) * kCUs;      // workgroups of a split: bounds the parts to 34 MB
    for (unsigned s = 1; s <= 16; ++s) {
      if (s > 1 && (stages < 2 * s || count * s > most)) break;
      const unsigned per = share(stages, s), splits = (stages + per - 1) / per;   // no empty split
      const double stage = (double)((count * splits + kCUs - 1) / kCUs) * c.shared;
      double us = ((double)per + fill) * (c.lone + cold > stage ? c.lone + cold : stage);
      if (splits > 1) us += reduce + 8e-6 / 4 * (double)splits * (double)M * (double)N;
      if (best.us == 0 || us < best.us) best = EdgePrice{us, {c.tile, (int)splits}};
    }
  }
  return best;
}
// Few columns of a large weight
bool weight_bound(int dtype, i64 M, i64 N, i64 K) { return N <= 32 && (double)M * (double)K * (dtype == POETX_F32 ? 4.0 : 2.0) > kLargeWeight; }
Plan dense_plan(int dtype, i64 M, i64 N, i64 K) {
  if (!weight_bound(dtype, M, N, K)) return edge_price(dtype, M, N, K).plan;
  const i64 count = tile_count(1, M, N, 32);
  if (count > 4 * kCUs) return Plan{TILE_32, 1};
  const unsigned depth = (unsigned)stage_depth(TILE_32, dtype == POETX_F32 ? 4 : 2), stages = ((unsigned)K + depth - 1) / depth;
  const unsigned four_each = 4 * kCUs / (unsigned)count, two_each = four_each / 2;     // workgroups of a tile for four and two on every CU
  const unsigned two = two_each < stages / 2 ? two_each : stages / 2, four = four_each < stages / 4 ? four_each : stages / 4, s = two > four ? two : four;
  if (s <= 1) return Plan{TILE_32, 1};
  const unsigned per = (stages + s - 1) / s;
  return Plan{TILE_32, (int)((stages + per - 1) / per)};
}
// Block gradients: the contraction is the token range, so a large tile with a split costs only its fp32 parts, while
// every halving of the tile side doubles the reads of both activations.  A split keeps 256 tokens, on the smallest tile two
// stages (one stage each: 1376 x 512, b = 64 step 93 -> 101 us).
Plan grad_plan(int dtype, int d, i64 N, int b) {
  const int nb = ceil_div(d, b);
  const size_t es = dtype == POETX_F32 ? 4 : 2;
  Plan p{TILE_32, 1};
  i64 most = N / (2 * stage_depth(TILE_32, es));
  int side = 32;
  for (const int t : {128, 64})
    if (b >= t && tile_count(nb, b, b, t) * (N / 256 > 1 ? N / 256 : 1) >= kCUs * 3 / 4) {
      p.tile = t == 128 ? TILE_128 : TILE_64;
      side = t;
      most = N / 256;
      break;
    }
  const i64 depth = stage_depth(p.tile, es), stages = (N + depth - 1) / depth;
  const i64 s = min64(2 * kCUs / tile_count(nb, b, b, side), most);
  if (s > 1) {
    const i64 per = (stages + s - 1) / s;
    p.splits = (int)((stages + per - 1) / per);
  }
  return p;
}

// ---- epilogues ---------------------------------------------------------------------------------
template <class T>
struct EpiStore {           // rows of a plain matrix
  T* out;
  i64 ld;
  int M, N;
  __device__ void operator()(int, int, int row, int col, const float (&v)[8]) const {
    if (row < M && col < N) store8(out + (i64)row * ld + col, v, N - col);
  }
};
struct EpiPartial {         // fp32 [split][batch][M][N]
  float* out;
  int M, N, batches;
  __device__ void operator()(int batch, int split, int row, int col, const float (&v)[8]) const {
    if (row < M && col < N) store8(out + (((i64)split * batches + batch) * M + row) * N + col, v, N - col);
  }
};
// Rows scattered through the permutation.  For bf16 blocks (stored as G - I) the identity part is added
// here in fp32 from the very row that gathered it; `valid` is the number of input columns, columns from
// there to `cols` are written as zeros.
template <class T, Load LOAD>
struct EpiScatter {
  T* out;
  const T* V;
  i64 ldo, ldv;
  const int32_t* perm;
  int b, d, valid, cols;
  __device__ void operator()(int batch, int, int row, int col, const float (&v)[8]) const {
    const int r = batch * b + row;
    if (row >= b || r >= d || col >= cols) return;
    const i64 at = perm[r];
    if constexpr (sizeof(T) == 2) {
      u32x4 x;
      if constexpr (LOAD == MASKED) x = mask_raw(load_raw(V + at * ldv, col, valid), col, valid, true);
      else x = load_branched(V + at * ldv, col, valid, true);
      float w[8];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        w[2 * e] = v[2 * e] + bf16_bits_to_float((uint16_t)(x[e] & 0xFFFF));
        w[2 * e + 1] = v[2 * e + 1] + bf16_bits_to_float((uint16_t)(x[e] >> 16));
      }
      store8(out + at * ldo + col, w, cols - col);
    } else {
      store8(out + at * ldo + col, v, cols - col);
    }
  }
};

// The same where V or out is token major (feature r of token c at c * ld + r): a few tokens, element by element.
template <class T, bool V_TM, bool OUT_TM>
struct EpiScatterTokens {
  T* out;
  const T* V;
  i64 ldo, ldv;
  const int32_t* perm;
  int b, d, valid, cols;
  __device__ void operator()(int batch, int, int row, int col, const float (&v)[8]) const {
    const int r = batch * b + row;
    if (row >= b || r >= d) return;
    const i64 at = perm[r];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int c = col + e;
      if (c >= cols) break;
      float x = v[e];
      if constexpr (sizeof(T) == 2) {
        if (c < valid) x += bf16_bits_to_float(V[V_TM ? c * ldv + at : at * ldv + c]);
        out[OUT_TM ? c * ldo + at : at * ldo + c] = (T)mm::pack2_bf16(x, 0.f);
      } else {
        out[OUT_TM ? c * ldo + at : at * ldo + c] = x;
      }
    }
  }
};

// out (M x N, row stride ld) = sum of the partials, in order
template <class T>
__global__ __launch_bounds__(256) void edge_reduce_kernel(const float* __restrict__ part, i64 total, int splits, T* __restrict__ out, int N, i64 ld) {
  const i64 e = ((i64)blockIdx.x * 256 + threadIdx.x) * 4;
  if (e >= total) return;
  float s[4] = {0.f, 0.f, 0.f, 0.f};
  if (e + 4 <= total && (total & 3) == 0) {
    for (int z = 0; z < splits; ++z) {
      const float4 p = *reinterpret_cast<const float4*>(part + z * total + e);
      s[0] += p.x; s[1] += p.y; s[2] += p.z; s[3] += p.w;
    }
  } else {
    for (int z = 0; z < splits; ++z)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (e + i < total) s[i] += part[z * total + e + i];
  }
  i64 row = e / N;
  int col = (int)(e - row * N);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (e + i < total) {
      if constexpr (sizeof(T) == 2) out[row * ld + col] = (T)mm::pack2_bf16(s[i], 0.f);
      else out[row * ld + col] = s[i];
    }
    if (++col == N) { col = 0; ++row; }
  }
}

// The same for two sums of whole vectors, n0 the number of workgroups of the first
struct ReduceSide {
  const float* part;
  float* out;
  i64 total;
  int splits;
};
__global__ __launch_bounds__(256) void edge_reduce_pair_kernel(ReduceSide s0, ReduceSide s1, int n0) {
  const bool second = (int)blockIdx.x >= n0;
  const ReduceSide s = second ? s1 : s0;
  const i64 e = ((i64)(blockIdx.x - (second ? n0 : 0)) * 256 + threadIdx.x) * 4;
  if (e >= s.total) return;
  float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int z = 0; z < s.splits; ++z) {
    const float4 p = *reinterpret_cast<const float4*>(s.part + z * s.total + e);
    v.x += p.x; v.y += p.y; v.z += p.z; v.w += p.w;
  }
  typedef float f4 __attribute__((ext_vector_type(4), aligned(4)));   // out may be the caller's
  *reinterpret_cast<f4*>(s.out + e) = f4{v.x, v.y, v.z, v.w};
}

template <class T>
void reduce(const float* part, i64 M, i64 N, int splits, T* out, i64 ld, hipStream_t st) {
  hipLaunchKernelGGL(edge_reduce_kernel<T>, dim3((unsigned)((M * N + 1023) / 1024)), dim3(256), 0, st, part, M * N, splits, out, (int)N, ld);
}

template <class T, bool A_K, class Epi>
void launch_slice_tile(SliceTile tile, const SliceArgs& g, const Epi& epi, i64 N, int splits, hipStream_t st) {
  if constexpr (sizeof(T) == 2 && !A_K) {
    if (tile == SLICES_64x32) return launch_slices<T, 64, 32, 4, 2, A_K>(g, epi, N, splits, st);
  }
  if (tile == SLICES_32) launch_slices<T, 32, 32, 8, 2, A_K>(g, epi, N, splits, st);
  else if (tile == SLICES_32x64) launch_slices<T, 32, 64, 4, 2, A_K>(g, epi, N, splits, st);
  else launch_slices<T, 64, 64, 4, 2, A_K>(g, epi, N, splits, st);
}
template <class T>
void dense_slices(const SlicePlan& p, int trans_w, const T* W, int n, int m, const T* act, i64 act_cols, T* out, i64 ld_out, i64 N, float* parts, hipStream_t st) {
  const int M = trans_w ? m : n, K = trans_w ? n : m;
  const SliceArgs g{W, act, m, act_cols, M, (int)act_cols, 0, slice_count(K, (int)sizeof(T)), 0};
  if (p.splits > 1) {
    const EpiPartial epi{parts, M, (int)N, 1};
    if (trans_w) launch_slice_tile<T, false>(p.tile, g, epi, N, p.splits, st);
    else launch_slice_tile<T, true>(p.tile, g, epi, N, p.splits, st);
    reduce<T>(parts, M, N, p.splits, out, ld_out, st);
  } else {
    const EpiStore<T> epi{out, ld_out, M, (int)N};
    if (trans_w) launch_slice_tile<T, false>(p.tile, g, epi, N, 1, st);
    else launch_slice_tile<T, true>(p.tile, g, epi, N, 1, st);
  }
}

template <class T>
void dense_t(int dtype, int trans_w, const T* W, int n, int m, const T* act, i64 ld_act, i64 act_cols, T* out, i64 ld_out, i64 N, void* ws,
             hipStream_t st) {
  const int M = trans_w ? m : n, K = trans_w ? n : m;
  if (slices_take(dtype, M, m, act_cols, K) && ld_act == act_cols && (((uintptr_t)W | (uintptr_t)act) & 15) == 0) {
    const SlicePlan sp = slice_plan(dtype, trans_w, M, act_cols, K);
    if (sp.tile != EDGE_TILES) return dense_slices(sp, trans_w, W, n, m, act, act_cols, out, ld_out, N, (float*)ws, st);
  }
  const Plan p = dense_plan(dtype, M, act_cols, K);
  Args g{};
  g.A = Op{W, m, 0, nullptr, n, m, 0, 0};
  g.B = Op{act, ld_act, 0, nullptr, K, (int)act_cols, 0, 0};   // whole vectors: columns from N on are not stored
  if (p.splits > 1) {
    const EpiPartial epi{(float*)ws, M, (int)N, 1};
    if (trans_w) launch<T, false, false, DENSE>(g, epi, 1, M, N, K, p, st);
    else launch<T, true, false, DENSE>(g, epi, 1, M, N, K, p, st);
    reduce<T>((const float*)ws, M, N, p.splits, out, ld_out, st);
  } else {
    const EpiStore<T> epi{out, ld_out, M, (int)N};
    if (trans_w) launch<T, false, false, DENSE>(g, epi, 1, M, N, K, p, st);
    else launch<T, true, false, DENSE>(g, epi, 1, M, N, K, p, st);
  }
}

template <class T, Load LOAD>
void apply_t(const T* V, i64 ldv, T* out, i64 ldo, int d, i64 cols, i64 cols_out, i64 plan_cols, const int32_t* perm, const T* blocks, int b,
             int trans, hipStream_t st) {
  const int nb = ceil_div(d, b);
  const Tile t = apply_tile(nb, b, plan_cols);
  Args g{};
  g.rpb = b;
  g.d = d;
  g.B = Op{V, ldv, 0, perm, b, (int)cols, 1, 0};
  const EpiScatter<T, LOAD> epi{out, V, ldo, ldv, perm, b, d, (int)cols, (int)cols_out};
  if constexpr (sizeof(T) == 2) {   // pairs (E, E^T): op(E) has contiguous rows either way
    g.A = Op{blocks + (trans ? (i64)b * b : 0), b, 2ll * b * b, nullptr, b, b, 1, 1};
    launch_apply<T, true, false, LOAD>(g, epi, nb, b, cols_out, b, t, st);
  } else {
    g.A = Op{blocks, b, (i64)b * b, nullptr, b, b, 1, 1};
    if (trans) launch_apply<T, false, false, LOAD>(g, epi, nb, b, cols_out, b, t, st);
    else launch_apply<T, true, false, LOAD>(g, epi, nb, b, cols_out, b, t, st);
  }
}

// A few tokens, V or out token major, on the smallest tile (see edge_apply_smallest_tile): what bounds these are the scattered
// two- and four-byte accesses, each on a cache line of its own, of which a few tokens have few.
template <class T, bool V_TM, bool OUT_TM>
void apply_tokens_t(const T* V, i64 ldv, T* out, i64 ldo, int d, i64 cols, i64 cols_out, const int32_t* perm, const T* blocks, int b, int trans,
                    hipStream_t st) {
  const int nb = ceil_div(d, b);
  Args g{};
  g.rpb = b;
  g.d = d;
  // a token-major V has its features (rows) one element and its tokens (columns) ldv elements apart
  g.B = Op{V, V_TM ? 1 : ldv, 0, perm, b, (int)cols, 1, 0, V_TM ? ldv : 1};
  const EpiScatterTokens<T, V_TM, OUT_TM> epi{out, V, ldo, ldv, perm, b, d, (int)cols, (int)cols_out};
  if constexpr (sizeof(T) == 2) {
    g.A = Op{blocks + (trans ? (i64)b * b : 0), b, 2ll * b * b, nullptr, b, b, 1, 1};
    launch_apply_32<T, true, false, V_TM ? STRIDED : BRANCHED>(g, epi, nb, b, cols_out, b, st);
  } else {
    g.A = Op{blocks, b, (i64)b * b, nullptr, b, b, 1, 1};
    if (trans) launch_apply_32<T, false, false, V_TM ? STRIDED : BRANCHED>(g, epi, nb, b, cols_out, b, st);
    else launch_apply_32<T, true, false, V_TM ? STRIDED : BRANCHED>(g, epi, nb, b, cols_out, b, st);
  }
}

// block gradients as plan.splits parts at `parts`
template <class T>
Args grad_args(const GradProblem& q, int b) {
  Args g{};
  g.rpb = b;
  g.d = q.d;
  // A row's tail in one load where a padded row has the columns for it: they are zeros, and no stage starts past N (4090 masked element by
  // element cost nothing, but 55 tokens of 1536 x 1536, b = 256: whole backward 111.3 -> 108.7 us).
  const i64 whole = (q.N + 7) / 8 * 8;
  g.A = Op{q.U, q.ldu, 0, q.perm, b, (int)min64(q.cols_u, whole), 1, 0};
  g.B = Op{q.V, q.ldv, 0, q.perm, b, (int)min64(q.cols_v, whole), 1, 0};
  return g;
}
template <class T>
void grad_t(const Plan& p, const GradProblem& q, int b, hipStream_t st) {
  const int nb = ceil_div(q.d, b);
  launch<T, true, true, GRAD>(grad_args<T>(q, b), EpiPartial{q.parts, b, b, nb}, nb, b, b, q.N, p, st);
}
template <class T>
void grad_pair_t(const Plan& p0, const Plan& p1, const GradProblem& q0, const GradProblem& q1, int b, hipStream_t st) {
  const int n0 = ceil_div(q0.d, b), n1 = ceil_div(q1.d, b);
  launch_pair<T, true, true>(grad_args<T>(q0, b), grad_args<T>(q1, b), EpiPartial{q0.parts, b, b, n0}, EpiPartial{q1.parts, b, b, n1},
                             Problem{n0, b, b, q0.N}, Problem{n1, b, b, q1.N}, p0, p1, st);
}

}  // namespace

// Which of the two kernels it is depends on the pointers' alignment as well, which a query does not see: the parts of either.  Every linear call asks,
// so each product is priced once.
size_t edge_dense_workspace_bytes(int dtype, int trans_w, int n, int m, i64 act_cols, bool aligned) {
  const i64 M = trans_w ? m : n, K = trans_w ? n : m;
  const bool bound = weight_bound(dtype, M, act_cols, K);
  const EdgePrice e = bound ? EdgePrice{0, dense_plan(dtype, M, act_cols, K)} : edge_price(dtype, M, act_cols, K);
  int splits = e.plan.splits;
  if (aligned && slices_take(dtype, M, m, act_cols, K)) {
    const SlicePlan s = slice_plan(dtype, trans_w, M, act_cols, K, bound ? nullptr : &e);
    if (s.tile != EDGE_TILES && s.splits > splits) splits = s.splits;
  }
  return splits > 1 ? (size_t)splits * M * act_cols * sizeof(float) : 0;
}

void edge_dense(int dtype, int trans_w, const void* W, int n, int m, const void* act, i64 ld_act, i64 act_cols, void* out, i64 ld_out, i64 N,
                void* ws, hipStream_t st) {
  if (dtype == POETX_F32)
    dense_t<float>(dtype, trans_w, (const float*)W, n, m, (const float*)act, ld_act, act_cols, (float*)out, ld_out, N, ws, st);
  else
    dense_t<uint16_t>(dtype, trans_w, (const uint16_t*)W, n, m, (const uint16_t*)act, ld_act, act_cols, (uint16_t*)out, ld_out, N, ws, st);
}

void edge_apply_left(int dtype, const void* V, i64 ldv, void* out, i64 ldo, int d, i64 cols, i64 cols_out, i64 plan_cols, const int32_t* perm,
                     const void* blocks, int b, int transpose_G, hipStream_t st) {
  if (dtype == POETX_F32)
    apply_t<float, BRANCHED>((const float*)V, ldv, (float*)out, ldo, d, cols, cols_out, plan_cols, perm, (const float*)blocks, b, transpose_G, st);
  else if (cols >= 8 && cols % 8 != 0)   // tails, in rows that hold a vector (see Load)
    apply_t<uint16_t, MASKED>((const uint16_t*)V, ldv, (uint16_t*)out, ldo, d, cols, cols_out, plan_cols, perm, (const uint16_t*)blocks, b, transpose_G, st);
  else
    apply_t<uint16_t, BRANCHED>((const uint16_t*)V, ldv, (uint16_t*)out, ldo, d, cols, cols_out, plan_cols, perm, (const uint16_t*)blocks, b, transpose_G, st);
}

bool edge_apply_smallest_tile(int d, i64 plan_cols, int b) { return apply_tile(ceil_div(d, b), b, plan_cols) == TILE_32; }

void edge_apply_tokens(int dtype, const void* V, i64 ldv, bool v_tm, void* out, i64 ldo, bool out_tm, int d, i64 cols, i64 cols_out,
                       const int32_t* perm, const void* blocks, int b, int transpose_G, hipStream_t st) {
  if (dtype == POETX_F32) {
    auto f = v_tm ? apply_tokens_t<float, true, false> : apply_tokens_t<float, false, true>;
    f((const float*)V, ldv, (float*)out, ldo, d, cols, cols_out, perm, (const float*)blocks, b, transpose_G, st);
  } else {
    auto f = v_tm ? apply_tokens_t<uint16_t, true, false> : apply_tokens_t<uint16_t, false, true>;
    f((const uint16_t*)V, ldv, (uint16_t*)out, ldo, d, cols, cols_out, perm, (const uint16_t*)blocks, b, transpose_G, st);
  }
}

size_t edge_blockgrad_parts_bytes(int dtype, int d, i64 N, int b) {
  return (size_t)grad_plan(dtype, d, N, b).splits * ceil_div(d, b) * b * b * sizeof(float);
}

int edge_blockgrad_parts(int dtype, const GradProblem& q, int b, hipStream_t st) {
  const Plan p = grad_plan(dtype, q.d, q.N, b);
  if (dtype == POETX_F32) grad_t<float>(p, q, b, st);
  else grad_t<uint16_t>(p, q, b, st);
  return p.splits;
}

void edge_blockgrad_parts_pair(int dtype, const GradProblem& q0, const GradProblem& q1, int b, int* n0, int* n1, hipStream_t st) {
  const Plan p0 = grad_plan(dtype, q0.d, q0.N, b), p1 = grad_plan(dtype, q1.d, q1.N, b);
  *n0 = p0.splits;
  *n1 = p1.splits;
  if (p0.tile != p1.tile) {
    edge_blockgrad_parts(dtype, q0, b, st);
    edge_blockgrad_parts(dtype, q1, b, st);
  } else if (dtype == POETX_F32) {
    grad_pair_t<float>(p0, p1, q0, q1, b, st);
  } else {
    grad_pair_t<uint16_t>(p0, p1, q0, q1, b, st);
  }
}

namespace {
template <class T, Load LOAD>
void apply_pair_t(Tile t, const T* V, i64 ldv, T* out, i64 ldo, i64 cols, i64 cols_out, const T* blocks, const Plan& p0, const Plan& p1, const GradProblem& q0,
                  const GradProblem& q1, int b, hipStream_t st) {
  constexpr int D = 128 / (int)sizeof(T);
  const int n0 = ceil_div(q0.d, b), n1 = ceil_div(q1.d, b);
  Args g{};
  g.rpb = b;
  g.d = q1.d;
  g.B = Op{V, ldv, 0, q1.perm, b, (int)cols, 1, 0};
  g.A = Op{blocks, b, (sizeof(T) == 2 ? 2ll : 1ll) * b * b, nullptr, b, b, 1, 1};
  const EpiScatter<T, LOAD> epi{out, V, ldo, ldv, q1.perm, b, q1.d, (int)cols, (int)cols_out};
  const Problem qa{n1, b, cols_out, b}, g0{n0, b, b, q0.N}, g1{n1, b, b, q1.N};
  const EpiPartial e0{q0.parts, b, b, n0}, e1{q1.parts, b, b, n1};
  auto go = [&](auto launch) { launch(g, epi, qa, grad_args<T>(q0, b), grad_args<T>(q1, b), e0, e1, g0, g1, p0.splits, p1.splits, st); };
  constexpr bool M = LOAD == MASKED;
  using E = EpiScatter<T, LOAD>;
  // the shapes of launch_apply
  if (t == TILE_64) go(launch_apply_pair<T, 64, D, 2, 4, M, E, EpiPartial>);
  else if (b > D) go(launch_apply_pair<T, 32, 2 * D, 1, 4, M, E, EpiPartial>);
  else go(launch_apply_pair<T, 32, D, 1, sizeof(T) == 2 ? 2 : 4, M, E, EpiPartial>);
}
}  // namespace

// Both on tiles that one launch holds: few of the apply, so that they do not fill the chip for long, and with the gradients' (whose blocks may be very many) no more than one grid
// dimension takes.  us, two launches without the gap between them / one: fp32 256 x 256, b = 32, 512 tokens
// 3.9 + 5.4 / 5.6; 1024 x 768, b = 64, 1001 tokens 5.9 + 10.7 / 12.1; bf16 1376 x 512, b = 64, 1024 tokens 4.3 + 5.9 / 6.5.  Whole backward calls of 220 random small layers: 13 % less on
// average, 1 % more at worst (apply tiles up to four per CU, 16 - 4096 tokens).
bool edge_apply_joins_blockgrads(int dtype, int d_apply, i64 plan_cols, int d0, int d1, i64 N, int b) {
  const Tile t = apply_tile(ceil_div(d_apply, b), b, plan_cols);
  const Plan p0 = grad_plan(dtype, d0, N, b), p1 = grad_plan(dtype, d1, N, b);
  if (t == TILE_128 || p0.tile != TILE_32 || p1.tile != TILE_32) return false;
  const i64 apply = tile_count(ceil_div(d_apply, b), b, plan_cols, t == TILE_64 ? 64 : 32);
  return apply <= 4 * kCUs && apply + tile_count(ceil_div(d0, b), b, b, 32) * p0.splits + tile_count(ceil_div(d1, b), b, b, 32) * p1.splits <= kGridRow;
}

// dX = R dA (out = op(blocks) V on the rows of q1's side) and both sides' block gradients
void edge_apply_blockgrad_parts(int dtype, const void* V, i64 ldv, void* out, i64 ldo, i64 cols, i64 cols_out, i64 plan_cols, const void* blocks, const GradProblem& q0,
                                const GradProblem& q1, int b, int* n0, int* n1, hipStream_t st) {
  const Plan p0 = grad_plan(dtype, q0.d, q0.N, b), p1 = grad_plan(dtype, q1.d, q1.N, b);
  *n0 = p0.splits;
  *n1 = p1.splits;
  const Tile t = apply_tile(ceil_div(q1.d, b), b, plan_cols);
  if (dtype == POETX_F32) apply_pair_t<float, BRANCHED>(t, (const float*)V, ldv, (float*)out, ldo, cols, cols_out, (const float*)blocks, p0, p1, q0, q1, b, st);
  else if (cols >= 8 && cols % 8 != 0) apply_pair_t<uint16_t, MASKED>(t, (const uint16_t*)V, ldv, (uint16_t*)out, ldo, cols, cols_out, (const uint16_t*)blocks, p0, p1, q0, q1, b, st);
  else apply_pair_t<uint16_t, BRANCHED>(t, (const uint16_t*)V, ldv, (uint16_t*)out, ldo, cols, cols_out, (const uint16_t*)blocks, p0, p1, q0, q1, b, st);
}

size_t edge_blockgrad_workspace_bytes(int dtype, int d, i64 N, int b) {
  const int splits = grad_plan(dtype, d, N, b).splits;
  return splits > 1 ? (size_t)splits * ceil_div(d, b) * b * b * sizeof(float) : 0;
}

// Both sides: one launch (where their tiles are the same) and one that adds the parts of both.  Parts of a side lie behind each other in ws, whole vectors (b * b a multiple of four).
size_t edge_blockgrad_pair_workspace_bytes(int dtype, int d0, int d1, i64 N, int b) {
  return align256(edge_blockgrad_workspace_bytes(dtype, d0, N, b)) + align256(edge_blockgrad_workspace_bytes(dtype, d1, N, b));
}
void edge_blockgrad_pair(int dtype, GradProblem q0, GradProblem q1, int b, float* dG0, float* dG1, void* ws, hipStream_t st) {
  const bool split0 = grad_plan(dtype, q0.d, q0.N, b).splits > 1, split1 = grad_plan(dtype, q1.d, q1.N, b).splits > 1;
  q0.parts = split0 ? (float*)ws : dG0;
  q1.parts = split1 ? (float*)((char*)ws + align256(edge_blockgrad_workspace_bytes(dtype, q0.d, q0.N, b))) : dG1;
  int n0 = 1, n1 = 1;
  edge_blockgrad_parts_pair(dtype, q0, q1, b, &n0, &n1, st);
  const ReduceSide s0{q0.parts, dG0, split0 ? (i64)ceil_div(q0.d, b) * b * b : 0, n0}, s1{q1.parts, dG1, split1 ? (i64)ceil_div(q1.d, b) * b * b : 0, n1};
  const int w0 = ceil_div(s0.total, 1024), w1 = ceil_div(s1.total, 1024);
  if (w0 + w1 > 0) hipLaunchKernelGGL(edge_reduce_pair_kernel, dim3((unsigned)(w0 + w1)), dim3(256), 0, st, s0, s1, w0);
}

void edge_blockgrad(int dtype, GradProblem q, int b, float* dG, void* ws, hipStream_t st) {
  const bool split = grad_plan(dtype, q.d, q.N, b).splits > 1;
  q.parts = split ? (float*)ws : dG;
  const int n = edge_blockgrad_parts(dtype, q, b, st);
  if (split) reduce<float>((const float*)ws, (i64)ceil_div(q.d, b) * b, b, n, dG, b, st);
}

}  // namespace poetx
