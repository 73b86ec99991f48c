// Fused permutation-gather + block-diagonal product + permutation-scatter on bf16
// activations (Eq. 2 with Eq. 5 and Eq. 7; mm1 / mm3 of Eq. 10 and their input
// gradients):
//     out[pi[j*b + i], t] = V[pi[j*b + i], t] + sum_l op(E_j)(i, l) * V[pi[j*b + l], t]
// with E = G - I, so neither the permutation nor the orthogonal matrix is ever
// materialised and the identity part of G is carried exactly.
//
// The stage is HBM bound (b/2 flop per byte), so the kernels are organised around the memory stream: the
// gathered rows of a block are contiguous runs of tokens, pass through LDS once, are multiplied from there with
// transposing reads and leave with the same row pattern (scatter by the same index map).  Blocks are stored as
// the pair (E, E^T) so that op(E)(i, .) is always a contiguous row.
#include "edge_gemm.h"

namespace poetx {
namespace {

using mm::bf16x8;
using mm::floatx16;
using mm::short4v;
using mm::short8v;

constexpr int SBN256 = 128, SBN = 64;   // tokens of a tile: of long streams at b = 256, and elsewhere

// ---------------------------------------------------------------------------------------
// One persistent workgroup per (block, 256-row slice of it, token range).
//   * 8 waves; wave w owns 32 output rows of the slice for computing and storing.
//   * those rows of op(E_j) stay in registers as matrix-core fragments for the whole range
//     (B/16 k steps x 4 VGPRs), so the block operand is read once per workgroup.
//   * token tiles of BN go from HBM straight into a 2-stage LDS ring (global_load_lds, all B
//     rows of the block gathered through the permutation, XOR-swizzled chunks, no bank
//     conflicts); the tile of the next step is in flight while the current one is multiplied.
//   * the identity part of G is applied as one exact extra MFMA per k step that covers the
//     wave's own rows (1.0 * x accumulates exactly in fp32), so nothing is re-read.
//   * results leave from registers: a lane owns one row and 4 consecutive tokens (8-byte
//     packed stores), scattered through the same index map that gathered them.
// b = 256: one slice.  b = 512: two slices per block (the block operand of
// a whole block does not fit the register file); the two workgroups of a
// block read the same token tiles, the second read being served by L2 / Infinity Cache.
// Tiles of 64 tokens (one 128-byte line of a row) fill the chip from half the tokens that 128 take and start sooner; long streams are read and written from
// memory in 256-byte pieces of a row (b = 256, us in a layer, 64 / 128 tokens a tile: 4096 features, 4096 tokens 18.4 / 19.6, 16384 70.9 / 63.6 = 4.2 TB/s;
// 14336 features, 16384 tokens 223 / 207).
template <int B, int BN>
__global__ __launch_bounds__(512) void apply_left_stream_kernel(const uint16_t* __restrict__ V,
                                                                 uint16_t* __restrict__ out, i64 ld,
                                                                 const int32_t* __restrict__ perm,
                                                                 const uint16_t* __restrict__ blocks, int trans, int tiles,
                                                                 int tiles_per_wg, int paired_chunks) {
  constexpr int MSPLIT = B / 256, TN = BN / 32, KS = B / 16;
  constexpr int STAGE_BYTES = B * BN * 2;
  constexpr int CPR = BN / 8;                        // 16-byte chunks per row
  constexpr int RPI = 64 / CPR;                      // rows filled by one direct-to-LDS instruction
  constexpr int IPW = STAGE_BYTES / 1024 / 8;        // such instructions per wave per stage
  extern __shared__ __attribute__((aligned(1024))) char ring[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // Which (block, slice, token range).  With two slices per block (paired_chunks > 0, one-dimensional
  // grid) the two workgroups that read the same token tiles get ids 8 apart: consecutive ids go to the
  // 8 XCDs in turn, so the pair shares one L2 and the tiles cross the fabric once.
  int j = blockIdx.y, slice = blockIdx.x % MSPLIT, chunk = blockIdx.x / MSPLIT;
  if (MSPLIT == 2 && paired_chunks > 0) {
    const int id = blockIdx.x, pair = (id >> 4) * 8 + (id & 7);
    slice = (id >> 3) & 1;
    j = pair / paired_chunks;
    chunk = pair % paired_chunks;
  }
  const int first = chunk * tiles_per_wg;
  const int T = tiles - first < tiles_per_wg ? tiles - first : tiles_per_wg;
  if (T <= 0) return;
  const i64 tok0 = (i64)first * BN;
  const int32_t* pm = perm + (i64)j * B;
  const int li = lane & 31, h = lane >> 5;
  const uint32_t ring_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)ring;

  // direct-to-LDS instruction s of this wave fills chunk slots [(IPW*w+s)*64, +64) of a stage:
  // row k = (IPW*w+s)*RPI + lane/CPR, chunk position lane%CPR -> logical chunk through the swizzle.
  i64 goff[IPW];
#pragma unroll
  for (int s = 0; s < IPW; ++s) {
    const int k = (wave * IPW + s) * RPI + lane / CPR;
    const int c = mm::kx_unchunk<BN>(lane % CPR, k);
    goff[s] = (i64)pm[k] * ld + tok0 + c * 8;
  }
  auto issue = [&](int t) {
    const uint32_t stage = ring_base + (t & 1) * STAGE_BYTES + wave * IPW * 1024;
#pragma unroll
    for (int s = 0; s < IPW; ++s) mm::dma16(V + goff[s] + (i64)t * BN, stage + s * 1024);
  };
  issue(0);

  // block operand fragments (rows of op(E_j) are contiguous in the stored pair)
  const int row_own = slice * 256 + wave * 32 + li;
  const uint16_t* Eb = blocks + ((i64)j * 2 + (trans ? 1 : 0)) * B * B + (i64)row_own * B + 8 * h;
  bf16x8 fa[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) fa[ks] = *reinterpret_cast<const bf16x8*>(Eb + ks * 16);
  // identity fragments for the two k steps that cover the wave's own 32 rows
  bf16x8 fi[2];
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int e = 0; e < 8; ++e) fi[u][e] = (li == u * 16 + 8 * h + e) ? (__bf16)1.0f : (__bf16)0.0f;
  const int own_kpair = slice * 8 + wave;  // k steps 2*own_kpair and 2*own_kpair + 1

  // LDS byte offsets of this lane's token fragments at k step 0
  int fragB[TN];
  {
    const int q = lane >> 4, i = lane & 15;
    const int k = 8 * (q >> 1) + (i >> 2);
#pragma unroll
    for (int c2 = 0; c2 < TN; ++c2) {
      const int c = c2 * 4 + 2 * (q & 1) + ((i & 3) >> 1);
      fragB[c2] = k * (BN * 2) + 16 * mm::kx_chunk<BN>(c, k) + 8 * (i & 1);
    }
  }
  // Results leave through a per-wave staging area behind the ring (32 rows x 64 tokens = 4 KB): the
  // wave writes a 64-token half of its tile there in accumulator order and reads it back with 8
  // consecutive lanes on one row, so that every global store instruction writes whole 128-byte row
  // segments (scattered through the same index map that gathered the rows).  Only the wave itself
  // touches its area, so its own lgkmcnt wait is all the synchronisation this needs.
  constexpr int NH = TN / 2;                          // 64-token halves of a tile
  char* stg = ring + 2 * STAGE_BYTES + wave * 4096;
  // write side: row li, chunk (8 tokens) cl*4 + 2p + h of the half, XOR-swizzled by the row pair
  const int stg_w = li * 128 + 16 * (h ^ ((li >> 1) & 7));
  // read side / stores: rows (lane >> 3) + 8 i, chunk lane & 7
  i64 soff[4];
  int stg_r[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = (lane >> 3) + 8 * i;
    soff[i] = (i64)pm[slice * 256 + wave * 32 + r] * ld + tok0 + 8 * (lane & 7);
    stg_r[i] = r * 128 + 16 * ((lane & 7) ^ ((r >> 1) & 7));
  }

  // The stores of a tile are issued one iteration late, right after the next barrier: by the
  // following barrier both those stores and the loads of the next tile are old, so a plain
  // vmcnt(0) there waits for nothing that is not already due (loads and stores share one counter
  // and may retire out of order with respect to each other).
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  u32x4 pend[NH * 4];
  auto flush = [&](int t) {
#pragma unroll
    for (int hf = 0; hf < NH; ++hf)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        *reinterpret_cast<u32x4*>(out + soff[i] + (i64)t * BN + hf * 64) = pend[hf * 4 + i];
  };
  for (int t = 0; t < T; ++t) {
    // tile t has landed and every wave is done reading the stage that tile t+1 overwrites: the
    // wait covers this wave's own LDS reads too (lgkmcnt), so the ring does not depend on where the
    // compiler places the MFMAs that consume them
    mm::wait_all_reads_and_barrier<0>();
    if (t > 0) flush(t - 1);
    if (t + 1 < T) issue(t + 1);
    const char* stage = ring + (t & 1) * STAGE_BYTES;
    auto load_tok = [&](bf16x8* fb, int ks) {
#pragma unroll
      for (int c = 0; c < TN; ++c) {
        const char* p = stage + fragB[c] + ks * 16 * (BN * 2);
        short4v lo = mm::lds_read_tr(p);
        short4v hi = mm::lds_read_tr(p + 4 * (BN * 2));
        short8v v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        fb[c] = __builtin_bit_cast(bf16x8, v);
      }
    };
    floatx16 acc[TN];
#pragma unroll
    for (int c = 0; c < TN; ++c)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[c][v] = 0.f;
    // identity part first (the two k steps that cover the wave's own rows: a wave-uniform LDS
    // address, no branch in the main loop), then the block operand with the token fragments of
    // the next k step always in flight under the MFMAs of the current one
    bf16x8 fo[2][TN], fb[2][TN];
    load_tok(fo[0], 2 * own_kpair);
    load_tok(fo[1], 2 * own_kpair + 1);
    load_tok(fb[0], 0);
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int c = 0; c < TN; ++c) acc[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fo[u][c], fi[u], acc[c], 0, 0, 0);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      if (ks + 1 < KS) load_tok(fb[(ks + 1) & 1], ks + 1);
#pragma unroll
      for (int c = 0; c < TN; ++c)
        acc[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[ks & 1][c], fa[ks], acc[c], 0, 0, 0);
    }
    // round; registers 4q..4q+3 hold tokens 8q + 4h + 0..3.  v_permlane32_swap exchanges the upper
    // lane half of its first operand with the lower half of its second, which leaves the lower lanes
    // with tokens 16p .. 16p+7 and the upper lanes with tokens 16p+8 .. 16p+15 of the 32-token
    // tile: 16-byte pieces, written to the staging area and read back row by row
#pragma unroll
    for (int hf = 0; hf < NH; ++hf) {
#pragma unroll
      for (int cl = 0; cl < 2; ++cl) {
        const int c = 2 * hf + cl;
        uint32_t w[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) w[e] = mm::pack2_bf16(acc[c][2 * e], acc[c][2 * e + 1]);
#pragma unroll
        for (int p = 0; p < 2; ++p) {
          typedef unsigned uint2v __attribute__((ext_vector_type(2)));
          const uint2v r0 = __builtin_amdgcn_permlane32_swap(w[4 * p], w[4 * p + 2], false, false);
          const uint2v r1 = __builtin_amdgcn_permlane32_swap(w[4 * p + 1], w[4 * p + 3], false, false);
          // chunk cl*4 + 2p + h: the XOR with the row pair commutes with adding the even part
          *reinterpret_cast<u32x4*>(stg + (stg_w ^ (16 * (cl * 4 + 2 * p)))) = u32x4{r0[0], r1[0], r0[1], r1[1]};
        }
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
      for (int i = 0; i < 4; ++i) pend[hf * 4 + i] = *reinterpret_cast<const u32x4*>(stg + stg_r[i]);
      if (hf + 1 < NH) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // read back before the area is rewritten
    }
  }
  flush(T - 1);
}

// Tiles per workgroup of `units` block slices with `tiles` token tiles each: the fewest tile times on 256 CUs, a workgroup's lead-in (indices, block operand, first
// tile) counted as three tiles.  (Measured, b = 256: 6 us and 1.7 a tile, 3.6 where all CUs share the memory; b = 512: 9.6 and 2.9, 4.3.)  Each count is tried up to
// 64, then steps of a 64th, so that with millions of tokens the search does not take longer than the launch.
int tiles_per_workgroup(i64 units, int tiles) {
  int per = tiles;
  i64 best = 0;
  for (int p = 1; p <= tiles; p += 1 + p / 64) {
    const i64 rounds = (units * ceil_div(tiles, p) + 255) / 256, cost = rounds * (p + 3);
    if (best == 0 || cost < best) { best = cost; per = p; }
    if (rounds == 1) break;   // longer ranges only cost more
  }
  return per;
}

// Chunks of long streams (128-token tiles): whole rounds of 256 workgroups of at least two tiles.
int stream_chunks(int slices, int tiles) {
  int best = 1;
  double best_eff = 0.0;
  for (int c = 1; c <= tiles; c *= 2) {
    if (tiles % c != 0 || tiles / c < 2) break;
    const double wgs = (double)slices * c;
    const double rounds = (double)(long long)((wgs + 255) / 256);
    const double eff = wgs / 256.0 / rounds;
    if (eff > best_eff + 1e-9) { best_eff = eff; best = c; }
  }
  return best;
}

template <int B, int BN>
void launch_apply_stream(const uint16_t* V, uint16_t* out, int d, i64 cols, i64 ld, const int32_t* perm,
                         const uint16_t* E, int trans, hipStream_t st) {
  constexpr size_t LDS = 2 * (size_t)B * BN * 2 + 8 * 4096;   // 2-stage ring + per-wave output staging
  constexpr int MSPLIT = B / 256;
  auto kern = apply_left_stream_kernel<B, BN>;
  // once per kernel instance; a function-local static is initialised exactly once, whichever thread gets there first
  static const bool configured =
      hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)LDS) == hipSuccess;
  (void)configured;
  const int nb = d / B, tiles = (int)(cols / BN);
  const int per = BN == 128 ? tiles / stream_chunks(nb * MSPLIT, tiles) : tiles_per_workgroup((i64)nb * MSPLIT, tiles), chunks = ceil_div(tiles, per);
  if (MSPLIT == 2 && ((i64)nb * chunks) % 8 == 0)
    hipLaunchKernelGGL(kern, dim3(chunks * MSPLIT * nb), dim3(512), LDS, st, V, out, ld, perm, E, trans, tiles, per, chunks);
  else
    hipLaunchKernelGGL(kern, dim3(chunks * MSPLIT, nb), dim3(512), LDS, st, V, out, ld, perm, E, trans, tiles, per, 0);
}

// ---------------------------------------------------------------------------------------
// The streaming kernel for token counts and row strides of any kind (V: nv columns, row stride ldv; out: no columns, row
// stride ldo; columns nv .. no - 1 of out are zeros).  Direct-to-LDS loads need aligned rows, so the tiles come through
// registers (element-aligned 16-byte loads, masked at the last column) -- the loads of tile t + 1 are in flight while
// tile t is multiplied and are written to the other LDS stage after it -- and the output pieces are stored element
// aligned.  Everything else is the kernel above at 64 tokens per tile (128 leave no registers for the staging).
// 8192 x 4090, b = 256: 43 us = 3.1 TB/s (128 x 128 edge tiles, which read rows twice and the block once per tile: 94 us;
// the aligned kernel at 4096 tokens: 27 us).
template <int B>
__global__ __launch_bounds__(512) void apply_left_ragged_kernel(const uint16_t* __restrict__ V, uint16_t* __restrict__ out, i64 ldv, i64 ldo,
                                                                 int nv, int no, const int32_t* __restrict__ perm,
                                                                 const uint16_t* __restrict__ blocks, int trans, int tiles, int tiles_per_wg) {
  constexpr int BN = 64, MSPLIT = B / 256, TN = BN / 32, KS = B / 16;
  constexpr int STAGE_BYTES = B * BN * 2;
  constexpr int CPR = BN / 8, RPI = 64 / CPR, IPW = STAGE_BYTES / 1024 / 8;
  extern __shared__ __attribute__((aligned(1024))) char ring[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j = blockIdx.y, slice = blockIdx.x % MSPLIT, chunk = blockIdx.x / MSPLIT;
  const int first = chunk * tiles_per_wg;
  const int T = tiles - first < tiles_per_wg ? tiles - first : tiles_per_wg;
  if (T <= 0) return;
  const int tok0 = first * BN;
  const int32_t* pm = perm + (i64)j * B;
  const int li = lane & 31, h = lane >> 5;

  i64 goff[IPW];
#pragma unroll
  for (int s = 0; s < IPW; ++s) goff[s] = (i64)pm[(wave * IPW + s) * RPI + lane / CPR] * ldv;
  const int gcol = tok0 + mm::kx_unchunk<BN>(lane % CPR, lane / CPR) * 8;   // the swizzle repeats after RPI rows
  edge::u32x4 stage_regs[IPW];
  // Whole tiles without masks, the last one masked on its way into LDS: where it is loaded that would wait for the loads (2048 x 5632, 1999
  // tokens, b = 256: 21.3 and 15.7 -> 20.5 and 12.8 us).  b = 512 has no registers for that: masked by branches around the loads (4001 tokens of 8192 x 3072,
  // forward 303 us so, 316 the other way).
  auto gload = [&](int t) {
    if constexpr (B == 512) {
#pragma unroll
      for (int s = 0; s < IPW; ++s) stage_regs[s] = edge::load_branched(V + goff[s], gcol + t * BN, nv, true);
    } else if (tile_inside(tok0 + t * BN, BN, nv)) {
#pragma unroll
      for (int s = 0; s < IPW; ++s) stage_regs[s] = edge::load16(V + goff[s] + gcol + t * BN);
    } else {
#pragma unroll
      for (int s = 0; s < IPW; ++s) stage_regs[s] = edge::load_raw(V + goff[s], gcol + t * BN, nv);
    }
  };
  auto lstore = [&](int t) {
    if (B != 512 && !tile_inside(tok0 + t * BN, BN, nv)) {
#pragma unroll
      for (int s = 0; s < IPW; ++s) stage_regs[s] = edge::mask_raw(stage_regs[s], gcol + t * BN, nv, true);
    }
    char* stage = ring + (t & 1) * STAGE_BYTES + wave * IPW * 1024 + lane * 16;
#pragma unroll
    for (int s = 0; s < IPW; ++s) *reinterpret_cast<edge::u32x4*>(stage + s * 1024) = stage_regs[s];
  };
  gload(0);

  const int row_own = slice * 256 + wave * 32 + li;
  const uint16_t* Eb = blocks + ((i64)j * 2 + (trans ? 1 : 0)) * B * B + (i64)row_own * B + 8 * h;
  bf16x8 fa[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) fa[ks] = *reinterpret_cast<const bf16x8*>(Eb + ks * 16);
  bf16x8 fi[2];
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int e = 0; e < 8; ++e) fi[u][e] = (li == u * 16 + 8 * h + e) ? (__bf16)1.0f : (__bf16)0.0f;
  const int own_kpair = slice * 8 + wave;

  int fragB[TN];
  {
    const int q = lane >> 4, i = lane & 15;
    const int k = 8 * (q >> 1) + (i >> 2);
#pragma unroll
    for (int c2 = 0; c2 < TN; ++c2) {
      const int c = c2 * 4 + 2 * (q & 1) + ((i & 3) >> 1);
      fragB[c2] = k * (BN * 2) + 16 * mm::kx_chunk<BN>(c, k) + 8 * (i & 1);
    }
  }
  char* stg = ring + 2 * STAGE_BYTES + wave * 4096;   // per-wave output staging, see the kernel above
  const int stg_w = li * 128 + 16 * (h ^ ((li >> 1) & 7));
  i64 soff[4];
  int stg_r[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = (lane >> 3) + 8 * i;
    soff[i] = (i64)pm[slice * 256 + wave * 32 + r] * ldo;
    stg_r[i] = r * 128 + 16 * ((lane & 7) ^ ((r >> 1) & 7));
  }
  const int scol = tok0 + 8 * (lane & 7);
  edge::u32x4 pend[4];
  auto flush = [&](int t) {
    const int col = scol + t * BN;
    if (no - col >= 8) {
#pragma unroll
      for (int i = 0; i < 4; ++i) *reinterpret_cast<edge::u32x4_a2*>(out + soff[i] + col) = pend[i];
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int e = 0; e < 7; ++e)
          if (col + e < no) out[soff[i] + col + e] = (uint16_t)(pend[i][e >> 1] >> (16 * (e & 1)));
    }
  };
  lstore(0);
  for (int t = 0; t < T; ++t) {
    // tile t is in LDS, and every wave is done reading the stage that tile t + 1 will overwrite
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (t + 1 < T) gload(t + 1);
    if (t > 0) flush(t - 1);
    const char* stage = ring + (t & 1) * STAGE_BYTES;
    auto load_tok = [&](bf16x8* fb, int ks) {
#pragma unroll
      for (int c = 0; c < TN; ++c) {
        const char* p = stage + fragB[c] + ks * 16 * (BN * 2);
        short4v lo = mm::lds_read_tr(p);
        short4v hi = mm::lds_read_tr(p + 4 * (BN * 2));
        short8v v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        fb[c] = __builtin_bit_cast(bf16x8, v);
      }
    };
    floatx16 acc[TN];
#pragma unroll
    for (int c = 0; c < TN; ++c)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[c][v] = 0.f;
    bf16x8 fo[2][TN], fb[2][TN];
    load_tok(fo[0], 2 * own_kpair);
    load_tok(fo[1], 2 * own_kpair + 1);
    load_tok(fb[0], 0);
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int c = 0; c < TN; ++c) acc[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fo[u][c], fi[u], acc[c], 0, 0, 0);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      if (ks + 1 < KS) load_tok(fb[(ks + 1) & 1], ks + 1);
#pragma unroll
      for (int c = 0; c < TN; ++c) acc[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[ks & 1][c], fa[ks], acc[c], 0, 0, 0);
    }
#pragma unroll
    for (int cl = 0; cl < TN; ++cl) {
      uint32_t w[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) w[e] = mm::pack2_bf16(acc[cl][2 * e], acc[cl][2 * e + 1]);
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        typedef unsigned uint2v __attribute__((ext_vector_type(2)));
        const uint2v r0 = __builtin_amdgcn_permlane32_swap(w[4 * p], w[4 * p + 2], false, false);
        const uint2v r1 = __builtin_amdgcn_permlane32_swap(w[4 * p + 1], w[4 * p + 3], false, false);
        *reinterpret_cast<edge::u32x4*>(stg + (stg_w ^ (16 * (cl * 4 + 2 * p)))) = edge::u32x4{r0[0], r1[0], r0[1], r1[1]};
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int i = 0; i < 4; ++i) pend[i] = *reinterpret_cast<const edge::u32x4*>(stg + stg_r[i]);
    if (t + 1 < T) lstore(t + 1);
  }
  flush(T - 1);
}

template <int B>
void launch_apply_ragged(const uint16_t* V, i64 ldv, i64 nv, uint16_t* out, i64 ldo, i64 no, int d, const int32_t* perm, const uint16_t* E,
                         int trans, hipStream_t st) {
  constexpr size_t LDS = 2 * (size_t)B * 64 * 2 + 8 * 4096;
  constexpr int MSPLIT = B / 256;
  auto kern = apply_left_ragged_kernel<B>;
  // once per kernel instance; a function-local static is initialised exactly once, whichever thread gets there first
  static const bool configured =
      hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)LDS) == hipSuccess;
  (void)configured;
  const int nb = d / B, tiles = ceil_div(no, 64);
  const int per = tiles_per_workgroup((i64)nb * MSPLIT, tiles);
  hipLaunchKernelGGL(kern, dim3(ceil_div(tiles, per) * MSPLIT, nb), dim3(512), LDS, st, V, out, ldv, ldo, (int)nv, (int)no, perm, E, trans, tiles, per);
}

}  // namespace

bool mfma_apply_left_supported(int d, i64 cols, i64 ld, int b) {
  if (d % b != 0 || ld % 8 != 0) return false;
  if (b == 256) return cols % SBN256 == 0;
  if (b == 512) return cols % SBN == 0;
  return false;
}

void mfma_apply_left(const void* V, void* out, int d, i64 cols, i64 ld, const int32_t* perm, const void* E, int b,
                     int transpose_G, hipStream_t st) {
  if (b == 512) {
    // A tile per workgroup and CUs to spare: the ragged kernel's loads through registers are there earlier (us, here / there: 512 features, 64 tokens 11.7 / 11.1, 2048, 1088 13.2 / 12.9; not with
    // every CU busy: 2048, 2048 14.6 / 15.0).  The same bits.
    if (d / 256 * (cols / SBN) < 256) return mfma_apply_left_ragged(V, ld, cols, out, ld, cols, d, perm, E, b, transpose_G, st);
    return launch_apply_stream<512, SBN>((const uint16_t*)V, (uint16_t*)out, d, cols, ld, perm, (const uint16_t*)E, transpose_G, st);
  }
  // By 64-token tiles per workgroup.  One or two: the ragged kernel's loads through registers are there a little earlier (us: 4096 features, 1024 tokens 10.4 / 9.5, 2048
  // 14.2 / 13.3, with 128-token tiles 14.6 and 16.7; 8192 features, 2048 tokens, four tiles, 21.7 / 23.4).  From eight on 128-token tiles (see the kernel).  All three sum in
  // the same order: the bits do not depend on the choice.
  const int per = tiles_per_workgroup(d / 256, (int)(cols / SBN));
  if (per <= 2) mfma_apply_left_ragged(V, ld, cols, out, ld, cols, d, perm, E, b, transpose_G, st);
  else if (per < 8 || cols % (2 * SBN256) != 0) launch_apply_stream<256, SBN>((const uint16_t*)V, (uint16_t*)out, d, cols, ld, perm, (const uint16_t*)E, transpose_G, st);
  else launch_apply_stream<256, SBN256>((const uint16_t*)V, (uint16_t*)out, d, cols, ld, perm, (const uint16_t*)E, transpose_G, st);
}

// The edge kernel reads the block operand once per tile and more than one workgroup reads a row, the streaming form starts with a chain
// of latencies (block operand, first tile).  us per apply of a ragged count, streaming / edge (back to back calls cost 8 us each at
// least): b = 256, d = 14336: 9.4 / 10.6 at 100 columns, 11.0 / 19.6 at 250, 12.3 / 23.5 at 300; d = 4096: 8.2 / 8.3, 8.8 / 9.3,
// 8.7 / 10.7.  b = 512, d = 14336: 16.5 / 16.4, 20.0 / 31.7, 20.1 / 38.3; d = 4096: 14.3 / 10.2, 14.5 / 14.1, 15.5 / 16.3; d = 1024:
// 14.0 / 9.1, 13.7 / 9.2, 14.0 / 10.3.  256 columns: at least as fast but for the few blocks of a small b = 512 side.
bool mfma_apply_left_ragged_supported(int d, i64 cols_out, int b) { return (b == 256 || b == 512) && d % b == 0 && cols_out >= 256; }

void mfma_apply_left_ragged(const void* V, i64 ldv, i64 cols, void* out, i64 ldo, i64 cols_out, int d, const int32_t* perm, const void* E, int b,
                            int transpose_G, hipStream_t st) {
  if (b == 256) launch_apply_ragged<256>((const uint16_t*)V, ldv, cols, (uint16_t*)out, ldo, cols_out, d, perm, (const uint16_t*)E, transpose_G, st);
  else launch_apply_ragged<512>((const uint16_t*)V, ldv, cols, (uint16_t*)out, ldo, cols_out, d, perm, (const uint16_t*)E, transpose_G, st);
}

}  // namespace poetx
