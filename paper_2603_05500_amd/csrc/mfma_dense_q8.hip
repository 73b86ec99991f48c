// Dense bf16 products on an INT8 base weight (Sec. 3.6, POET-XQ): the weight is dequantised on the
// fly inside the product, no high-precision copy of it is ever written to memory.
//   forward : B  (n x N) = W   A,   backward: dA (m x N) = W^T dB,   W[i][k] = scale[i] * q[i][k].
//
// Same persistent stream as the bf16 product (mfma_dense.hip: one wave per SIMD, 128 x 128 wave
// tiles, 32-deep stages through an LDS ring, one barrier per stage); only the weight operand takes
// another road into its ring slot.  Its 8-bit codes (8 KB per stage) and the scales the stage needs
// arrive by direct-to-LDS loads in a small side ring; two stages ahead of the multiplication (three and four ahead of it they are in flight) each
// wave converts exactly the bytes it loaded itself -- so its own vmcnt wait is all the
// synchronisation the side ring needs -- into bf16(scale * q) and writes them into the weight half
// of the stage's slot, in the layout the bf16 kernel uses.  The conversion (one cvt + one fma per
// element, rounded once to fp32 and once to bf16, i.e. bit for bit the stand-alone dequantiser)
// runs in the shadow of the MFMAs.
#include "mfma_dense_kernel.h"

namespace poetx {
namespace {

using dense::dma16g;
using dense::dma16g_s;
using dense::floatx4;
using mm::bf16x8;
using mm::short4v;
using mm::short8v;

constexpr int BM = 256, BN = 256, BK = 32, NW = 4, NS = 4, NQ = 3;
constexpr int A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2, STAGE_BYTES = A_BYTES + B_BYTES;
constexpr int Q_CODES = BM * BK;                 // 8 KB of codes per stage
constexpr int Q_SLOT = Q_CODES + 1024;           // + 256 floats of scales
constexpr int Q_BASE = NS * STAGE_BYTES;         // side ring behind the main ring
constexpr int LDS_BYTES = Q_BASE + NQ * Q_SLOT;  // 155648
constexpr int IPW = B_BYTES / 1024 / NW;         // 4 direct-to-LDS instructions per wave per stage for the activations
constexpr int QLOADS = 3;                        // per wave per stage: 2 x 16 bytes of codes per lane + 1 x 4 bytes of scale
constexpr int TM = BM / 32, TN = BN / 32, MF = TM * TN, GROUP = 4;
// At the barrier before stage kt the wave's own codes of stage kt+2 and everybody's activations of
// stage kt+1 must have landed.  Issue order: ... B(kt+1), Q(kt+2), B(kt+2), Q(kt+3), B(kt+3), Q(kt+4), barrier:
// the loads younger than Q(kt+2) are two activation stages and two code stages.
constexpr int VM_BOUND = 2 * IPW + 2 * QLOADS;
static_assert(NS * IPW + NQ * QLOADS < 64, "vmcnt range");

struct DenseQ8Args {
  const int8_t* Q;       // codes, n x m row major
  const float* scale;    // n
  const uint16_t* B;     // activations, K x N row major
  uint16_t* C;           // M x N row major
  i64 ldq, ldb, ldc;
  int tiles_m, tiles_n, ktiles;
  int splits;            // PARTS: the contraction in so many ranges of ktiles stages each, the first `longer` of them two longer (as in the bf16 product),
  int longer;
  float* parts;          // whose products go here in fp32, [split][M][N], instead of to C
};

__device__ inline void dma4s(const void* sbase, uint32_t voff, uint32_t lds_addr) {
  asm volatile("global_load_lds_dword %0, %1" ::"v"(voff), "s"(sbase), "{m0}"(lds_addr) : "memory");
}

// A_KMAJOR: forward (weight rows are output rows, contraction along a row).  Otherwise backward
// (weight rows are the contraction index).
template <bool A_KMAJOR, bool PARTS>
__global__ __launch_bounds__(256) void dense_q8_stream_kernel(DenseQ8Args g) {
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;

  const int T0 = g.tiles_m * g.tiles_n, T = PARTS ? T0 * g.splits : T0;
  const int G = gridDim.x;
  int wq = blockIdx.x;
  if ((G & 7) == 0) wq = (wq & 7) * (G >> 3) + (wq >> 3);
  const int n_my = wq < T ? (T - 1 - wq) / G + 1 : 0;
  if (n_my == 0) return;
  const int per_group = GROUP * g.tiles_n;
  auto tile_origin = [&](int ti, int& i0, int& j0, int& split) {
    int u = ti * G + wq;
    split = 0;
    if (PARTS) {
      split = u / T0;
      u -= split * T0;
    }
    const int first_m = (u / per_group) * GROUP;
    const int gsz = (g.tiles_m - first_m) < GROUP ? (g.tiles_m - first_m) : GROUP;
    i0 = (first_m + (u % per_group) % gsz) * BM;
    j0 = ((u % per_group) / gsz) * BN;
  };
  const int KT = g.ktiles + (PARTS && wq / T0 < g.longer ? 2 : 0);
  auto first_stage = [&](int split) { return PARTS ? dense::range_start(split, g.ktiles, g.longer) : 0; };
  const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;

  // ---- activations: as in the bf16 kernel
  uint32_t voffB[IPW];
#pragma unroll
  for (int s = 0; s < IPW; ++s) {
    const int slot = (wave * IPW + s) * 64 + lane;
    const int k = slot / (BN / 8), c = dense::kx16_chunk(slot % (BN / 8), k);
    voffB[s] = (uint32_t)((k * g.ldb + c * 8) * 2) - s * 1024;   // less the instruction offset of load s
  }
  const i64 stepB = (i64)BK * g.ldb * 2;
  const char* Bb;
  int b_tile = 0, b_kt = 0, b_slot = 0;
  auto b_base = [&](int ti) {
    int i0, j0, split;
    tile_origin(ti, i0, j0, split);
    Bb = (const char*)(g.B + j0) + first_stage(split) * stepB;
  };
  b_base(0);
  auto issue_b = [&](int s) { dma16g_s(s, Bb, voffB[s], lds_base + b_slot * STAGE_BYTES + A_BYTES + wave * IPW * 1024); };
  auto b_advance = [&]() {
    b_slot = b_slot + 1 == NS ? 0 : b_slot + 1;
    if (b_kt + 1 < KT) { ++b_kt; Bb += stepB; }
    else if (b_tile + 1 < n_my) { ++b_tile; b_kt = 0; b_base(b_tile); }
  };

  // ---- codes and scales.  Code instruction j of wave w fills 16-byte chunks [(2w+j)*64, +64) of the
  // side-ring slot; lane l owns chunk ch = (2w+j)*64 + l and converts it itself later.
  //   forward : the stage's codes are [256 rows][32 bytes]: row = ch >> 1, bytes 16 (ch & 1) ..
  //   backward: [32 k rows][256 bytes]: row = ch >> 4, bytes 16 (ch & 15) ..
  // The scale instruction of wave w fills floats [64w, 64w + 64) of the slot's scale area with the
  // scales of the rows its chunks belong to (forward: rows 64w + l; backward: k rows 8w + (l & 7)).
  uint32_t voffQ[2], voffS;
  int cvt_dst[2][2];     // byte offsets (inside the weight half of a stage) of the two bf16 chunks a code chunk becomes
  int cvt_scale[2];      // byte offset of the chunk's scale inside the slot
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int ch = (wave * 2 + j) * 64 + lane;
    if (A_KMAJOR) {
      const int r = ch >> 1, c = ch & 1;
      voffQ[j] = (uint32_t)(r * g.ldq + 16 * c) - j * 1024;
      cvt_dst[j][0] = r * 64 + 16 * dense::xk16_chunk(2 * c, r);
      cvt_dst[j][1] = r * 64 + 16 * dense::xk16_chunk(2 * c + 1, r);
      cvt_scale[j] = Q_CODES + 4 * r;
    } else {
      const int k = ch >> 4, c = ch & 15;
      voffQ[j] = (uint32_t)(k * g.ldq + 16 * c) - j * 1024;
      cvt_dst[j][0] = k * (BM * 2) + 16 * dense::kx16_chunk(2 * c, k);
      cvt_dst[j][1] = k * (BM * 2) + 16 * dense::kx16_chunk(2 * c + 1, k);
      cvt_scale[j] = Q_CODES + 4 * (64 * wave + (k - 8 * wave));
    }
  }
  voffS = A_KMAJOR ? (uint32_t)(4 * (64 * wave + lane)) : (uint32_t)(4 * (8 * wave + (lane & 7)));
  const i64 stepQ = A_KMAJOR ? (i64)BK : (i64)BK * g.ldq;          // bytes per stage along the contraction
  const char* Qb;
  const char* Sb;
  int q_tile = 0, q_kt = 0, q_slot = 0;
  auto q_base = [&](int ti) {
    int i0, j0, split;
    tile_origin(ti, i0, j0, split);
    Qb = (const char*)g.Q + (A_KMAJOR ? (i64)i0 * g.ldq : (i64)i0) + first_stage(split) * stepQ;
    Sb = (const char*)(g.scale + (A_KMAJOR ? i0 : first_stage(split) * BK));
  };
  q_base(0);
  auto issue_q = [&]() {
    const uint32_t slot = lds_base + Q_BASE + q_slot * Q_SLOT;
    dma16g<0>(Qb, voffQ[0], slot + wave * 2 * 1024);
    dma16g<1024>(Qb, voffQ[1], slot + wave * 2 * 1024);
    dma4s(Sb, voffS, slot + Q_CODES + wave * 256);
    q_slot = q_slot + 1 == NQ ? 0 : q_slot + 1;
    if (q_kt + 1 < KT) {
      ++q_kt;
      Qb += stepQ;
      if (!A_KMAJOR) Sb += BK * 4;
    } else if (q_tile + 1 < n_my) {
      ++q_tile;
      q_kt = 0;
      q_base(q_tile);
    }
  };
  // conversion side: which side-ring slot and which main-ring slot come next
  int c_qslot = 0, c_slot = 0;
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  struct Codes {
    u32x4 q[2];
    float s[2];
  };
  auto cvt_read = [&](Codes& c) {
    const char* slot = lds + Q_BASE + c_qslot * Q_SLOT;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      c.q[j] = *reinterpret_cast<const u32x4*>(slot + (wave * 2 + j) * 1024 + lane * 16);
      c.s[j] = *reinterpret_cast<const float*>(slot + cvt_scale[j]);
    }
    c_qslot = c_qslot + 1 == NQ ? 0 : c_qslot + 1;
  };
  // Conversion of chunk j in eight steps of two codes each (about six vector instructions: few enough
  // to sit between two MFMAs without delaying the second); after steps 3 and 7 one 16-byte chunk of
  // bf16 goes into the weight half of main-ring slot c_slot.
  uint32_t cvo[8];
  auto cvt_step = [&](const Codes& c, int j, int hw) {
    char* stage = lds + c_slot * STAGE_BYTES;
    const float s = c.s[j], off = -128.f * s;
    const uint32_t u = c.q[j][hw >> 1] ^ 0x80808080u;      // signed code + 128 as an unsigned byte
    const uint32_t b0 = (hw & 1) ? ((u >> 16) & 0xffu) : (u & 0xffu);
    const uint32_t b1 = (hw & 1) ? (u >> 24) : ((u >> 8) & 0xffu);
    // (u - 128) * s, rounded once: the fma adds the exact products u*s and -128*s
    cvo[hw] = mm::pack2_bf16(__builtin_fmaf((float)b0, s, off), __builtin_fmaf((float)b1, s, off));
    if (hw == 3) *reinterpret_cast<u32x4*>(stage + cvt_dst[j][0]) = u32x4{cvo[0], cvo[1], cvo[2], cvo[3]};
    if (hw == 7) *reinterpret_cast<u32x4*>(stage + cvt_dst[j][1]) = u32x4{cvo[4], cvo[5], cvo[6], cvo[7]};
  };
  auto cvt_write = [&](const Codes& c, int j) {
#pragma unroll
    for (int hw = 0; hw < 8; ++hw) cvt_step(c, j, hw);
  };
  auto cvt_done = [&]() { c_slot = c_slot + 1 == NS ? 0 : c_slot + 1; };

  // ---- fragments
  int fragA[TM], fragB[TN];
  {
    const int q = lane >> 4, i = lane & 15;
    const int k = 8 * q + (i >> 2);
#pragma unroll
    for (int a = 0; a < TM; ++a) {
      const int x0 = wm * (BM / 2) + a * 16;
      if (A_KMAJOR) {
        const int r = x0 + i;
        fragA[a] = r * 64 + 16 * dense::xk16_chunk(q, r);
      } else {
        fragA[a] = k * (BM * 2) + 16 * dense::kx16_chunk((x0 >> 3) + ((i & 3) >> 1), k) + 8 * (i & 1);
      }
    }
#pragma unroll
    for (int c2 = 0; c2 < TN; ++c2) {
      const int x0 = wn * (BN / 2) + c2 * 16;
      fragB[c2] = A_BYTES + k * (BN * 2) + 16 * dense::kx16_chunk((x0 >> 3) + ((i & 3) >> 1), k) + 8 * (i & 1);
    }
  }
  floatx4 acc[TM][TN];
#pragma unroll
  for (int a = 0; a < TM; ++a)
#pragma unroll
    for (int c = 0; c < TN; ++c) acc[a][c] = floatx4{0.f, 0.f, 0.f, 0.f};
  auto load_frag = [&](const char* p, bool kmajor, int row_bytes) -> bf16x8 {
    if (kmajor) return *reinterpret_cast<const bf16x8*>(p);
    const short4v lo = mm::lds_read_tr(p), hi = mm::lds_read_tr(p + 4 * row_bytes);
    const short8v v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8, v);
  };
  struct Frags {
    bf16x8 a[TM], b[TN];
  };
  auto load_piece = [&](Frags& f, const char* stage, int p) {   // in the order the MFMAs first need them
    if (p == 1) f.b[0] = load_frag(stage + fragB[0], false, BN * 2);
    else if (p <= TM) f.a[p ? p - 1 : 0] = load_frag(stage + fragA[p ? p - 1 : 0], A_KMAJOR, BM * 2);
    else f.b[p - TM] = load_frag(stage + fragB[p - TM], false, BN * 2);
  };

  // ---- prologue: codes of stages 0..2 and activations of stages 0, 1; stages 0 and 1 converted; then, in the order of the loop,
  // the activations of stages 2 and 3 and, into the slots that stages 0 and 1 have left, the codes of stages 3 and 4
  Codes cd;
  issue_q();
  issue_q();
  issue_q();
  auto issue_stage_b = [&]() {
#pragma unroll
    for (int s = 0; s < IPW; ++s) issue_b(s);
    b_advance();
  };
  issue_stage_b();
  issue_stage_b();
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    cvt_read(cd);
    cvt_write(cd, 0);
    cvt_write(cd, 1);
    cvt_done();
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // conversion reads done before their slots are refilled
  issue_stage_b();
  issue_q();
  issue_stage_b();
  issue_q();
  mm::wait_all_reads_and_barrier<VM_BOUND>();           // everybody's stage 0 is in place
  Frags F, Gf;
  int cslot = 0;
#pragma unroll
  for (int p = 0; p < TM + TN; ++p) load_piece(F, lds, p);

  const int q4 = lane >> 4, li = lane & 15;

  auto run = [&](auto WC) {
    constexpr int W = decltype(WC)::value;
    // stage kt from X; the fragments of the next one into Y; the activations of stage kt + NS into the slot of this one; the codes of stage kt + 2
    // converted into theirs, and those of stage kt + 5 into the side-ring slot they leave
    auto multiply = [&](const Frags& X, Frags& Y) {
      // every wave holds this stage in registers; the activations of the next stage and this wave's codes of the stage after it have
      // landed; the next stage's weights are converted
      mm::wait_all_reads_and_barrier<VM_BOUND>();
      const int nslot = cslot + 1 == NS ? 0 : cslot + 1;
      const char* nstage = lds + nslot * STAGE_BYTES;
#pragma unroll
      for (int i = 0; i < MF; ++i) {
        dense::mfma16(acc[i % TM][i / TM], X.b[i / TM], X.a[i % TM]);
        if (i == 0) cvt_read(cd);
        if (i % 3 == 1 && i / 3 < TM + TN) load_piece(Y, nstage, i / 3);
        if (i % 16 == 4 * W + 2) issue_b(i / 16);
        if (i >= 14 && i % 3 == 2 && (i - 14) / 3 < 16) cvt_step(cd, (i - 14) / 3 / 8, (i - 14) / 3 % 8);
        if (i == MF - 1) {
          cvt_done();
          b_advance();
          issue_q();
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      cslot = nslot;
    };
    for (int ti = 0; ti < n_my; ++ti) {
      for (int kt = 0; kt < KT; kt += 2) {
        multiply(F, Gf);
        multiply(Gf, F);
      }
      dense::settle(acc);
      int i0, j0, split;
      tile_origin(ti, i0, j0, split);
      if constexpr (PARTS) {
        float* P = g.parts + ((i64)split * (g.tiles_m * BM) + i0 + wm * (BM / 2) + li) * g.ldb + j0 + wn * (BN / 2) + 4 * q4;
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
          for (int c = 0; c < TN; ++c) {
            *reinterpret_cast<floatx4*>(P + (i64)(a * 16) * g.ldb + c * 16) = acc[a][c];
            acc[a][c] = floatx4{0.f, 0.f, 0.f, 0.f};
          }
      } else {
        uint16_t* Ct = g.C + (i64)(i0 + wm * (BM / 2) + li) * g.ldc + j0 + wn * (BN / 2) + 16 * (q4 & 1) + 8 * (q4 >> 1);
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
          for (int c = 0; c < TN; c += 2) {
            uint32_t o[4];
            dense::pack_pair(acc[a][c], acc[a][c + 1], o);
            acc[a][c] = floatx4{0.f, 0.f, 0.f, 0.f};
            acc[a][c + 1] = floatx4{0.f, 0.f, 0.f, 0.f};
            *reinterpret_cast<u32x4*>(Ct + (i64)a * 16 * g.ldc + c * 16) = u32x4{o[0], o[1], o[2], o[3]};
          }
      }
    }
  };
  switch (wave) {
    case 0: run(std::integral_constant<int, 0>{}); break;
    case 1: run(std::integral_constant<int, 1>{}); break;
    case 2: run(std::integral_constant<int, 2>{}); break;
    default: run(std::integral_constant<int, 3>{}); break;
  }
  mm::wait_vmcnt_and_barrier<0>();
}

int compute_units_q8() {
  static const int n = [] {
    int dev = 0, cu = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cu <= 0)
      cu = 256;
    return cu;
  }();
  return n;
}

template <bool A_KMAJOR, bool PARTS>
void launch_dense_q8(const DenseQ8Args& g, hipStream_t st) {
  auto kern = dense_q8_stream_kernel<A_KMAJOR, PARTS>;
  static const bool configured =
      hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES) == hipSuccess;
  (void)configured;
  const int T = g.tiles_m * g.tiles_n * g.splits, cus = compute_units_q8();
  hipLaunchKernelGGL(kern, dim3(T < cus || g.longer > 0 ? T : cus), dim3(256), LDS_BYTES, st, g);
}

}  // namespace

bool mfma_dense_q8_supported(int n, int m, i64 N) {
  // a stream of at least 3 stages per workgroup keeps the prologue simple; 32-bit lane offsets
  return mfma_dense_supported(n, m, N) && n >= 3 * BK && m >= 3 * BK;
}

// The contraction is split exactly where the bf16 product splits it, so that a layer gets the same bits either way.
void mfma_dense_q8(int trans_w, const void* Wq, int n, int m, const void* act, void* out, i64 N, void* ws, hipStream_t st) {
  const int M = trans_w ? m : n, K = trans_w ? n : m;
  DenseQ8Args g{};
  g.Q = (const int8_t*)Wq;
  g.scale = (const float*)((const char*)Wq + weight_q8_scale_offset(n, m));
  g.B = (const uint16_t*)act;
  g.C = (uint16_t*)out;
  g.ldq = m;
  g.ldb = N;
  g.ldc = N;
  g.tiles_m = M / BM;
  g.tiles_n = (int)(N / BN);
  g.splits = mfma_dense_splits(M, N, K);
  g.parts = (float*)ws;
  const dense::ContractionRange range = dense::contraction_ranges(K / BK, g.splits);
  g.ktiles = range.ktiles;
  g.longer = range.longer;
  if (g.splits > 1) {
    if (trans_w) launch_dense_q8<false, true>(g, st);
    else launch_dense_q8<true, true>(g, st);
    mfma_dense_reduce((const float*)ws, g.splits, M, N, out, N, N, st);
  } else {
    if (trans_w) launch_dense_q8<false, false>(g, st);
    else launch_dense_q8<true, false>(g, st);
  }
}

}  // namespace poetx
