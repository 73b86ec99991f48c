// Dense bf16 products of the POET-X linear layer on the matrix cores:
//   forward  (Eq. 10, mm2):       B  (n x N) = W   (n x m) * A  (m x N)
//   backward (Sec. 3.5, mm2 bwd): dA (m x N) = W^T (m x n) * dB (n x N)   -- no weight gradient
// W is row major n x m; activations are feature major (token index contiguous), so the
// activation operand (and W in the backward product) is contracted over its strided index and
// is read from LDS with the transposing load.
//
// The kernel is a persistent stream: one workgroup per CU, 4 waves (2 x 2, one per SIMD), each
// wave owning a 128 x 128 piece of a 256 x 256 output tile in 256 accumulator registers
// (v_mfma_f32_16x16x32_bf16, fp32; smaller tiles for products with few of them).  A workgroup walks its list of output tiles; the 32-deep
// operand stages of ALL its tiles form one stream that flows through a ring of 4 LDS stages
// (a fifth buys nothing measurable; its 32 KB stage the output instead),
// filled by direct-to-LDS loads issued that many stages ahead of the multiplication -- across tile
// boundaries, so a new tile starts multiplying the moment the previous one is rounded and stored.
// A wave multiplies a stage from registers while it reads the next one's fragments into a second set (128 registers for
// both), so the one barrier of a stage stands at its start, where every wave holds the stage: its slot is refilled at once.  Loads and
// fragment reads are pinned to fixed places between the MFMAs (each wave spreads its loads
// over different places), and the load addresses are a uniform base plus a per-lane offset that
// never changes, so the loop carries no vector address arithmetic and no branch.
//
// What bounds it is power: the clock falls until the chip keeps its limit, so what counts is energy per flop.  A loop of MFMAs alone on normally
// distributed operands sustains 2.04 PFLOP/s with 16 x 16 x 32 and 1.77 with 32 x 32 x 16 (an accumulator is read and written
// once per 32 of depth, not per 16; on zeros both reach 2.45).  The same stream on 32 x 32 x 16, before / now, us, sustained (smaller tiles without WIDE, see below): forward 4096 x 4096 x 16384 413 / 374,
// 14336 x 4096 x 16384 1420 / 1290; backward 400 / 369, 1405 / 1270; tiles of 256 x 128, 4096 x 4096 x 2048: 67 / 64.7 and 62.8 / 59; of 128 x 128, 2048 x 5632 x 2048:
// 51.8 / 50.9 and 50.8 / 49.
#pragma once
#include <type_traits>

#include "mfma_gemm.h"

namespace poetx {
namespace dense {


using mm::bf16x8;
typedef float floatx4 __attribute__((ext_vector_type(4)));
using mm::short4v;
using mm::short8v;

constexpr int BK = 32, NW = 4;
constexpr int GROUP = 4;                         // tile rows walked together

// Output tile and ring of one instance.  256 x 256 with 4 stages is the fast one (32 bytes of operands per cycle and CU);
// 256 x 128 (48 bytes) and 128 x 128 (64 bytes, what the L2 can deliver at best) exist for products with too few large
// tiles for the chip; their stages are shorter, so the ring is deeper.
template <int BM_, int BN_, int NS_>
struct Tile {
  static constexpr int BM = BM_, BN = BN_, NS = NS_;
  static constexpr int A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2, STAGE_BYTES = A_BYTES + B_BYTES;
  static constexpr int TM = BM / 32, TN = BN / 32;       // 16 x 16 MFMA tiles of a wave (2 x 2 waves)
  static constexpr int MF = TM * TN;                     // MFMAs of a stage
  // MFMAs per fragment read: the four waves' reads take up to half of the time of a stage's MFMAs in LDS (256 x 256; three quarters on 256 x 128, all of it
  // on 128 x 128); bunched, they would hold up the MFMAs behind them (256 x 256, backward, one / two / three: 391 / 382 / 379 us)
  static constexpr int RS = MF / (TM + TN) < 3 ? MF / (TM + TN) : 3;
  static constexpr int OUT_BYTES = TN / 4 * 4096;        // per-wave output staging: 32-row x 64-column pieces
  static constexpr int LDS_BYTES = NS * STAGE_BYTES + NW * OUT_BYTES;
  static constexpr int IPWA = A_BYTES / 1024 / NW;       // direct-to-LDS instructions per wave per operand per stage
  static constexpr int IPWB = B_BYTES / 1024 / NW;
  static constexpr int LPT = IPWA + IPWB;                // loads per stage per wave
  static_assert(NS * LPT < 64, "vmcnt range");
  static constexpr int DS = MF / LPT;                    // MFMAs per load
  static_assert(IPWA <= 4 && IPWB <= 4 && DS >= 1, "dma16g_s covers groups of four loads");
  static_assert(RS >= 1 && (TM + TN) * RS <= MF, "the next stage's fragments fit under this one's MFMAs");
  static_assert(LDS_BYTES <= 160 * 1024, "LDS of a CU");
};
typedef Tile<256, 256, 4> Tile256;        // 128 + 32 = 160 KB: the whole LDS of a CU
typedef Tile<256, 128, 6> Tile256x128;    // 144 + 16 KB
typedef Tile<128, 128, 8> Tile128;        // 128 + 16 KB

struct DenseArgs {
  const uint16_t* A;     // A_KMAJOR: M x K row major (lda = K stride); else K x M
  const uint16_t* B;     // K x N row major
  uint16_t* C;           // M x N row major
  i64 lda, ldb, ldc;
  int tiles_m, tiles_n, ktiles;   // ktiles counts 32-deep stages; even
  int cols;              // RAGGED: columns of C that exist; its rows need element alignment only
  int splits;            // PARTS: the contraction in so many ranges of ktiles stages each ...
  int longer;            // ... the first so many of them two stages longer (then a workgroup has one tile), see ContractionRange, ...
  float* parts;          // ... whose products go here in fp32, [split][M][N], instead of to C
};

// A contraction of `stages` in ranges: whole pairs of stages, as the streams multiply them two at a time
struct ContractionRange {
  int ktiles, longer;
};
inline ContractionRange contraction_ranges(int stages, int splits) { return ContractionRange{stages / 2 / splits * 2, stages / 2 % splits}; }
__device__ inline int range_start(int split, int ktiles, int longer) { return split * ktiles + 2 * (split < longer ? split : longer); }

// ---- swizzled tile layouts for 16 x 16 x 32 fragments (16-byte chunks) ----------------------------
// [x][k] tile: 4 chunks per row.  A 16-byte read serves 16 lanes at a time: lanes 0-3, 12-15, 20-23 and 24-27 (rows 0-3 and 12-15 of chunk c, 4-7 and 8-11 of
// chunk c + 1), then 4-11, 16-19 and 28-31, and the upper half the same way.  The four row groups of each get four positions.
__device__ inline int xk16_chunk(int c, int row) {
  const int x = (row >> 2) & 3;
  return c ^ (((x ^ (x >> 1)) & 1) << 1 | x >> 1);
}
// [k][x] tile.  A transposing read touches 4 consecutive k rows x 2 chunks per 16 lanes, rows 8 further down in the next 16: the k row
// spreads the former over 8 positions, its bit 3 puts the latter into the other 128 bytes.
__device__ inline int kx16_chunk(int c, int k) { return c ^ (2 * (k & 3)) ^ (((k >> 3) & 1) << 3); }

// c += a b on 16 x 16 x 32, in place.  Inline asm: the compiler gives the builtin's result other registers than its addend and then moves accumulators around
// (up to 300 spills here).  Its operands are loaded by code the compiler sees, which also inserts their waits; before the accumulators
// are read by anything but another of these, settle() lets the last of them finish.
__device__ __forceinline__ void mfma16(floatx4& c, const bf16x8& a, const bf16x8& b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
}
template <int TM, int TN>
__device__ __forceinline__ void settle(floatx4 (&c)[TM][TN]) {
  // the last TM products went to the last column of tiles; the others are at least TM products old
  static_assert(TM == 4 || TM == 8, "accumulator rows of a wave");
  constexpr int L = TN - 1;
  if constexpr (TM == 8)
    asm volatile("s_nop 15\n\ts_nop 3" : "+a"(c[0][L]), "+a"(c[1][L]), "+a"(c[2][L]), "+a"(c[3][L]), "+a"(c[4][L]), "+a"(c[5][L]), "+a"(c[6][L]), "+a"(c[7][L]));
  else
    asm volatile("s_nop 15\n\ts_nop 3" : "+a"(c[0][L]), "+a"(c[1][L]), "+a"(c[2][L]), "+a"(c[3][L]));
}

// Two neighbouring tiles' accumulators of a row (columns 4 (lane >> 4) .. + 3 of each) as eight consecutive bf16 columns per lane: 8 (lane >> 5) .. + 7 of
// the first tile in the even groups of 16 lanes, of the second in the odd ones.
__device__ __forceinline__ void pack_pair(const floatx4& x, const floatx4& y, uint32_t (&o)[4]) {
  typedef unsigned uint2v __attribute__((ext_vector_type(2)));
  const uint2v r0 = __builtin_amdgcn_permlane16_swap(mm::pack2_bf16(x[0], x[1]), mm::pack2_bf16(y[0], y[1]), false, false);
  const uint2v r1 = __builtin_amdgcn_permlane16_swap(mm::pack2_bf16(x[2], x[3]), mm::pack2_bf16(y[2], y[3]), false, false);
  o[0] = r0[0];
  o[1] = r1[0];
  o[2] = r0[1];
  o[3] = r1[1];
}

// 16 bytes per lane from (uniform base + per-lane byte offset + OFF) straight into LDS at
// lds_group + OFF + 16 * lane: the instruction offset moves the LDS address and the global address
// alike, so the per-lane offsets of a group of loads are biased by -OFF and the whole group shares
// one value of M0 (written once by the compiler, which tracks it as an operand).  Completion is
// tracked by hand through vmcnt.
template <int OFF>
__device__ inline void dma16g(const void* sbase, uint32_t voff, uint32_t lds_group) {
  asm volatile("global_load_lds_dwordx4 %0, %1 offset:%2" ::"v"(voff), "s"(sbase), "n"(OFF), "{m0}"(lds_group) : "memory");
}
// load s of a wave's group of up to four (s is a constant wherever this is called)
__device__ inline void dma16g_s(int s, const void* sbase, uint32_t voff, uint32_t lds_group) {
  switch (s) {
    case 0: dma16g<0>(sbase, voff, lds_group); break;
    case 1: dma16g<1024>(sbase, voff, lds_group); break;
    case 2: dma16g<2048>(sbase, voff, lds_group); break;
    default: dma16g<3072>(sbase, voff, lds_group); break;
  }
}

// DIAG bit 3: counts of this workgroup's second tile, per wave: [0] core cycles of its main loop, [1] of its
// output, [2] the main loop again in ticks of the constant 100 MHz counter (cycles / ticks = the clock the
// CU ran at); [3] ticks from the wave's start to its end.
static __device__ long long g_diag_cycles[4][4 * 256];

// DIAG (measurement builds only; the library instantiates DIAG = 0): bit 0 stops the direct-to-LDS loads
// after the prologue, bit 1 stops the fragment reads inside the loop, bit 2 keeps the load addresses on
// the first stage of the first tile (all loads hit in cache) -- the results are then wrong,
// bit 3 (harmless to the result) records the cycle counts above --
// every address stays what it was, and the timing shows what the loads or the reads cost.
// What a tile's epilogue writes: bf16 rows of C, the same with masked columns and element alignment, or fp32 parts.
enum Out { OUT_WHOLE = 0, OUT_RAGGED = 1, OUT_PARTS = 2 };
// OUT_RAGGED: the last tiles of a row reach past the columns of C (B is padded to whole tiles, C is not).
template <bool A_KMAJOR, Out OUT = OUT_WHOLE, int DIAG = 0, class C = Tile256>
__global__ __launch_bounds__(256) void dense_stream_kernel(DenseArgs g) {
  constexpr int BM = C::BM, BN = C::BN, NS = C::NS, A_BYTES = C::A_BYTES, STAGE_BYTES = C::STAGE_BYTES, OUT_BYTES = C::OUT_BYTES;
  constexpr int IPWA = C::IPWA, IPWB = C::IPWB, LPT = C::LPT, TM = C::TM, TN = C::TN, MF = C::MF, RS = C::RS, DS = C::DS;
  // WIDE: rows of a K-major A come 64 deep, whole 128-byte lines.  Two stages share a unit of A, which arrives in two halves of its rows, one per stage and one
  // stage later than B's tile of the same number (a unit is needed as a whole, and its slot is free, when its first stage is): the last half is in flight for NS - 3 stages, so
  // the ring has to be deep.  With 64-byte pieces every line is asked for twice; us, forward, weights from memory, 64 / 128 bytes:
  // 256 x 128 tiles, 4096 x 4096 x 2048 78.7 / 62; 128 x 128, 2048 x 5632 x 2048 69.5 / 55.
  constexpr bool WIDE = A_KMAJOR && NS >= 6;
  constexpr int A_STRIDE = WIDE ? A_BYTES : STAGE_BYTES, B_STRIDE = WIDE ? C::B_BYTES : STAGE_BYTES, B_BASE = WIDE ? NS * A_BYTES : A_BYTES;
  static_assert(!WIDE || NS % 2 == 0, "whole units");
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  long long t_start = 0;
  if (DIAG & 8) t_start = __builtin_amdgcn_s_memrealtime();

  // ---- this workgroup's tiles.  Workgroups go to the 8 XCDs round robin; in every step of
  // gridDim.x tiles each XCD takes a contiguous run of the tile order (GROUP tile rows walked
  // together), so the tiles an XCD works on at a time share operand panels in its L2.
  const int T0 = g.tiles_m * g.tiles_n;
  const int T = OUT == OUT_PARTS ? T0 * g.splits : T0;   // one contraction range after the other
  const int G = gridDim.x;
  int wq = blockIdx.x;
  if ((G & 7) == 0) wq = (wq & 7) * (G >> 3) + (wq >> 3);
  const int n_my = wq < T ? (T - 1 - wq) / G + 1 : 0;
  if (n_my == 0) return;
  const int per_group = GROUP * g.tiles_n;
  auto tile_origin = [&](int ti, int& i0, int& j0, int& split) {
    int u = ti * G + wq;
    split = 0;
    if (OUT == OUT_PARTS) {
      split = u / T0;
      u -= split * T0;
    }
    const int first_m = (u / per_group) * GROUP;
    const int gsz = (g.tiles_m - first_m) < GROUP ? (g.tiles_m - first_m) : GROUP;
    i0 = (first_m + (u % per_group) % gsz) * BM;
    j0 = ((u % per_group) / gsz) * BN;
  };

  // per-lane byte offsets of the direct-to-LDS loads (the same for every stage and tile), less the
  // instruction offset s * 1024 of load s (never negative: load s starts 16 s rows, or 2 s rows of at
  // least 256 elements, into the tile).
  // Instruction (wave, s) of IPW per operand fills LDS chunk slots [(wave*IPW + s)*64, +64) of the operand's part of
  // a stage; the lane's slot decides, through the inverse swizzle, which global chunk it fetches.
  uint32_t voffA[IPWA], voffB[IPWB];
#pragma unroll
  for (int s = 0; s < IPWA; ++s) {
    const int slot = (wave * IPWA + s) * 64 + lane;
    if (WIDE) {
      const int r = slot >> 3, c = (slot & 7) ^ ((r >> 1) & 7);
      voffA[s] = (uint32_t)((r * g.lda + c * 8) * 2) - s * 1024;
    } else if (A_KMAJOR) {
      const int r = slot >> 2, c = xk16_chunk(slot & 3, r);
      voffA[s] = (uint32_t)((r * g.lda + c * 8) * 2) - s * 1024;
    } else {
      const int k = slot / (BM / 8), c = kx16_chunk(slot % (BM / 8), k);
      voffA[s] = (uint32_t)((k * g.lda + c * 8) * 2) - s * 1024;
    }
  }
#pragma unroll
  for (int s = 0; s < IPWB; ++s) {
    const int slot = (wave * IPWB + s) * 64 + lane;
    const int k = slot / (BN / 8), c = kx16_chunk(slot % (BN / 8), k);
    voffB[s] = (uint32_t)((k * g.ldb + c * 8) * 2) - s * 1024;
  }
  const i64 stepA = A_KMAJOR ? (i64)BK * 2 : (i64)BK * g.lda * 2;
  const i64 stepB = (i64)BK * g.ldb * 2;
  const int KT = g.ktiles + (OUT == OUT_PARTS && wq / T0 < g.longer ? 2 : 0);
  const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;

  // ---- issue side of the stream: runs NS stages ahead of the multiplication, across tiles.  An, Bn: where the tile after the one in issue
  // starts, so that moving on is a choice between two values.  Past the last stage of the last tile the stream fetches that tile
  // from its start again: the number of loads in flight -- and with it the vmcnt bound of the barrier -- never changes.
  const char *Ab, *Bb, *An, *Bn;
  int ikt = 0, islot = 0, iah = 0, iaslot = 0;      // iah, iaslot: WIDE, half of a unit in issue and where it goes
  const i64 half_rows = (i64)(BM / 2) * g.lda * 2;
  auto tile_base = [&](int ti, const char*& a, const char*& b) {
    int i0, j0, split;
    tile_origin(ti < n_my ? ti : n_my - 1, i0, j0, split);
    const int first = OUT == OUT_PARTS ? range_start(split, g.ktiles, g.longer) : 0;
    a = (const char*)(g.A + (A_KMAJOR ? (i64)i0 * g.lda : (i64)i0)) + first * stepA;
    b = (const char*)(g.B + j0) + first * stepB;
  };
  tile_base(0, Ab, Bb);
  tile_base(1, An, Bn);
  bool loads_on = true;   // DIAG bit 0 switches it off after the prologue
  auto issue_a = [&](int s) { if (!(DIAG & 1) || loads_on) dma16g_s(s, Ab, voffA[s], lds_base + (WIDE ? iaslot : islot) * A_STRIDE + wave * IPWA * 1024); };
  auto issue_b = [&](int s) { if (!(DIAG & 1) || loads_on) dma16g_s(s, Bb, voffB[s], lds_base + islot * B_STRIDE + B_BASE + wave * IPWB * 1024); };
  auto issue_advance = [&]() {
    islot = islot + 1 == NS ? 0 : islot + 1;
    if (DIAG & 4) return;   // every stage re-fetches the first one: the loads stay, their misses go
    const bool last = ikt + 1 == KT;
    ikt = last ? 0 : ikt + 1;
    if (!WIDE) Ab = last ? An : Ab + stepA;
    Bb = last ? Bn : Bb + stepB;
  };
  auto a_half_advance = [&](bool second) {      // WIDE: from half `second` of a unit to the next
    iaslot = iaslot + 1 == NS ? 0 : iaslot + 1;
    const bool last = iah + 1 == KT;
    iah = last ? 0 : iah + 1;
    if (!second) Ab += half_rows;
    else Ab = last ? An : Ab + (2 * stepA - half_rows);
  };

  // ---- LDS byte offsets of this lane's fragments inside a stage: row (column) lane & 15 of a 16-wide piece, k = 8 (lane >> 4) .. + 7
  int fragA[TM], fragB[TN];
  {
    const int q = lane >> 4, i = lane & 15;
    const int k = 8 * q + (i >> 2);
#pragma unroll
    for (int a = 0; a < TM; ++a) {
      const int x0 = wm * (BM / 2) + a * 16;
      if (WIDE) {
        const int r = x0 + i;
        fragA[a] = r * 128 + 16 * (q ^ ((r >> 1) & 7));      // of a unit's first stage; the second's chunks are 4 further, bit 2 of the position
      } else if (A_KMAJOR) {
        const int r = x0 + i;
        fragA[a] = r * 64 + 16 * xk16_chunk(q, r);
      } else {
        fragA[a] = k * (BM * 2) + 16 * kx16_chunk((x0 >> 3) + ((i & 3) >> 1), k) + 8 * (i & 1);
      }
    }
#pragma unroll
    for (int c2 = 0; c2 < TN; ++c2) {
      const int x0 = wn * (BN / 2) + c2 * 16;
      fragB[c2] = B_BASE + k * (BN * 2) + 16 * kx16_chunk((x0 >> 3) + ((i & 3) >> 1), k) + 8 * (i & 1);
    }
  }

  floatx4 acc[TM][TN];
#pragma unroll
  for (int a = 0; a < TM; ++a)
#pragma unroll
    for (int c = 0; c < TN; ++c) acc[a][c] = floatx4{0.f, 0.f, 0.f, 0.f};

  auto load_frag = [&](const char* p, bool kmajor, int row_bytes) -> bf16x8 {
    if (kmajor) return *reinterpret_cast<const bf16x8*>(p);
    const short4v lo = mm::lds_read_tr(p), hi = mm::lds_read_tr(p + 4 * row_bytes);   // the swizzle is the same 4 rows further down
    const short8v v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8, v);
  };
  struct Frags {
    bf16x8 a[TM], b[TN];
  };
  // piece p of a stage's fragments, in the order the MFMAs first need them: A0 B0 A1 .. A(TM-1) B1 .. B(TN-1)
  auto load_piece = [&](Frags& f, int slot, bool odd, int p) {      // odd: the second stage of a unit
    const char* sa = lds + (WIDE && odd ? slot - 1 : slot) * A_STRIDE;
    const char* sb = lds + slot * B_STRIDE;
    if (p == 1) f.b[0] = load_frag(sb + fragB[0], false, BN * 2);
    else if (p <= TM) f.a[p ? p - 1 : 0] = load_frag(sa + (WIDE && odd ? fragA[p ? p - 1 : 0] ^ 64 : fragA[p ? p - 1 : 0]), A_KMAJOR, BM * 2);
    else f.b[p - TM] = load_frag(sb + fragB[p - TM], false, BN * 2);
  };

  // ---- prologue: stages 0 .. NS-1 (WIDE: the halves of A up to NS-2), in the order of the loop
#pragma unroll
  for (int t = 0; t < NS; ++t) {
    if (!WIDE || t > 0) {
#pragma unroll
      for (int s = 0; s < IPWA; ++s) issue_a(s);
      if (WIDE) a_half_advance(t % 2 == 0);      // half t - 1
    }
#pragma unroll
    for (int s = 0; s < IPWB; ++s) issue_b(s);
    issue_advance();
  }
  mm::wait_vmcnt_and_barrier<WIDE ? (NS - 3) * LPT + IPWB : (NS - 1) * LPT>();   // stage 0 (its unit) has landed
  Frags F, Gf;
  int cslot = 0;
#pragma unroll
  for (int p = 0; p < TM + TN; ++p) load_piece(F, 0, false, p);

  if (DIAG & 2) {   // the loop reads no fragments: both sets come from the first stage
#pragma unroll
    for (int p = 0; p < TM + TN; ++p) load_piece(Gf, 0, false, p);
  }
  loads_on = false;
  const int q4 = lane >> 4, li = lane & 15;

  // The body is instantiated once per wave: wave W issues its loads W quarters of the way from one to the next, so the four waves
  // do not hand the memory pipeline a load in the same place.
  auto run = [&](auto WC) {
    constexpr int W = decltype(WC)::value;
    // stage kt from X; the fragments of the next stage (the next tile's first one after the last one of this tile) into Y; stage kt + NS to issue
    auto multiply = [&](const Frags& X, Frags& Y, auto ODD) {
      constexpr bool odd = decltype(ODD)::value;       // this stage is the second of a unit
      // Every wave holds this stage in registers (lgkmcnt(0)) and the next one has landed: stages up to kt + NS - 1 are issued, so at
      // most NS - 2 of them may be in flight.  Stores of a finished tile share the counter and only make this wait stricter.
      // WIDE, a new unit next: its second half was the first thing issued NS - 3 stages ago.
      mm::wait_all_reads_and_barrier<WIDE && odd ? (NS - 4) * LPT + IPWB : (NS - 2) * LPT>();
      const int nslot = cslot + 1 == NS ? 0 : cslot + 1;
#pragma unroll
      for (int i = 0; i < MF; ++i) {
        // the operands go in swapped, so the accumulator tile is transposed: a lane owns one output row and four consecutive columns
        mfma16(acc[i % TM][i / TM], X.b[i / TM], X.a[i % TM]);
        if (i % RS == 0 && i / RS < TM + TN && !(DIAG & 2)) load_piece(Y, nslot, !odd, i / RS);
        if (i % DS == W * DS / 4 && i / DS < LPT) {
          if (i / DS < IPWA) issue_a(i / DS);
          else issue_b(i / DS - IPWA);
        }
        if (i == MF - 1) {
          issue_advance();
          if (WIDE) a_half_advance(!odd);      // half kt + NS - 1
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      cslot = nslot;
    };
    for (int ti = 0; ti < n_my; ++ti) {
      // the tile after the one in issue, which is NS stages ahead: that of stage NS of this tile
      if (ti > 0 || KT == NS) {      // KT >= 8 >= NS
        const char* unused;
        tile_base(ti + (KT > NS ? 1 : 2), An, Bn);
        if (WIDE && KT == NS) tile_base(ti + 1, An, unused);      // A is a stage behind, in this tile still
      }
      long long tc0 = 0, tc1 = 0, tr0 = 0, tr1 = 0;
      if ((DIAG & 8) && ti == 1) {
        tc0 = __builtin_readcyclecounter();
        tr0 = __builtin_amdgcn_s_memrealtime();
      }
      for (int kt = 0; kt < KT; kt += 2) {
        multiply(F, Gf, std::false_type{});
        multiply(Gf, F, std::true_type{});
      }
      if ((DIAG & 8) && ti == 1) {
        tc1 = __builtin_readcyclecounter();
        tr1 = __builtin_amdgcn_s_memrealtime();
      }
      // ---- tile done: round to bf16 and store, clear the accumulators.  The accumulator layout gives a
      // lane 4 consecutive columns of its row per 16-column tile; swapping two neighbouring tiles' between lane groups
      // (v_permlane16_swap: the odd groups of 16 lanes of its first operand against the even ones of its second)
      // makes that 8 columns = 16 bytes.  All workgroups finish their tiles together: the burst drains twice as fast when
      // every instruction writes whole 128-byte lines.  So the wave passes its piece through LDS, 32 rows
      // x 64 columns at a time (rows XOR-swizzled in 16-byte chunks, conflict free both ways), and reads
      // it back with 8 lanes per row.
      settle(acc);
      int i0, j0, split;
      tile_origin(ti, i0, j0, split);
      if constexpr (OUT == OUT_PARTS) {
        // fp32 parts: 16 columns of a row per instruction and row, 64 bytes
        float* P = g.parts + ((i64)split * (g.tiles_m * BM) + i0 + wm * (BM / 2) + li) * g.ldb + j0 + wn * (BN / 2) + 4 * q4;
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
          for (int c = 0; c < TN; ++c) {
            *reinterpret_cast<floatx4*>(P + (i64)(a * 16) * g.ldb + c * 16) = acc[a][c];
            acc[a][c] = floatx4{0.f, 0.f, 0.f, 0.f};
          }
      } else {
        typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
        char* stg = lds + NS * STAGE_BYTES + wave * OUT_BYTES;
        uint16_t* Cw = g.C + (i64)(i0 + wm * (BM / 2)) * g.ldc + j0 + wn * (BN / 2);
#pragma unroll
        for (int a = 0; a < TM / 2; ++a) {
#pragma unroll
          for (int a2 = 0; a2 < 2; ++a2) {
            const int row = a2 * 16 + li;
#pragma unroll
            for (int c = 0; c < TN; c += 2) {
              uint32_t o[4];
              pack_pair(acc[2 * a + a2][c], acc[2 * a + a2][c + 1], o);   // columns 8 (q4 >> 1) .. + 7 of tile c + (q4 & 1)
              acc[2 * a + a2][c] = floatx4{0.f, 0.f, 0.f, 0.f};
              acc[2 * a + a2][c + 1] = floatx4{0.f, 0.f, 0.f, 0.f};
              const int ch = ((c & 3) + (q4 & 1)) * 2 + (q4 >> 1);         // 16-byte chunk of the 64-column piece
              *reinterpret_cast<u32x4*>(stg + (c >> 2) * 4096 + row * 128 + 16 * (ch ^ ((row >> 1) & 7))) = u32x4{o[0], o[1], o[2], o[3]};
            }
          }
          asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // this wave's own writes; the area is private to it
#pragma unroll
          for (int cp = 0; cp < TN / 4; ++cp)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const int r = (lane >> 3) + 8 * i, ch = lane & 7;
              const u32x4 o = *reinterpret_cast<const u32x4*>(stg + cp * 4096 + r * 128 + 16 * (ch ^ ((r >> 1) & 7)));
              uint16_t* at = Cw + (i64)(a * 32 + r) * g.ldc + cp * 64 + ch * 8;
              if constexpr (OUT == OUT_RAGGED) {
                typedef uint32_t u32x4_a2 __attribute__((ext_vector_type(4), aligned(2)));
                const int left = g.cols - (j0 + wn * (BN / 2) + cp * 64 + ch * 8);
                if (left >= 8) {
                  *reinterpret_cast<u32x4_a2*>(at) = o;
                } else {
#pragma unroll
                  for (int e = 0; e < 7; ++e)
                    if (e < left) at[e] = (uint16_t)(o[e >> 1] >> (16 * (e & 1)));
                }
              } else {
                *reinterpret_cast<u32x4*>(at) = o;
              }
            }
        }
      }
      if ((DIAG & 8) && ti == 1 && lane == 0 && blockIdx.x < 256) {
        g_diag_cycles[0][blockIdx.x * 4 + W] = tc1 - tc0;
        g_diag_cycles[1][blockIdx.x * 4 + W] = __builtin_readcyclecounter() - tc1;
        g_diag_cycles[2][blockIdx.x * 4 + W] = tr1 - tr0;
      }
    }
  };
  switch (wave) {
    case 0: run(std::integral_constant<int, 0>{}); break;
    case 1: run(std::integral_constant<int, 1>{}); break;
    case 2: run(std::integral_constant<int, 2>{}); break;
    default: run(std::integral_constant<int, 3>{}); break;
  }
  mm::wait_vmcnt_and_barrier<0>();   // the re-fetched stages land before the LDS is released
  if ((DIAG & 8) && lane == 0 && blockIdx.x < 256) g_diag_cycles[3][blockIdx.x * 4 + wave] = __builtin_amdgcn_s_memrealtime() - t_start;
}


}  // namespace dense
}  // namespace poetx
