// Cayley-Neumann series and its backward on the matrix cores (Sec. 3.4, Eq. 8-9),
// batched over the blocks of one side, for block sides that do not fit on chip (b = 512).
//
// Every b x b product runs as bf16 x bf16 -> fp32 on the batched tile kernel; the dominant terms enter in fp32 in its
// epilogue.  A launch costs 20 us or so however small (512-deep contraction, fill, drain, epilogue), so the
// recurrences are chosen for few launches, and for little fp32 traffic between them: from 32 blocks on a launch fills the chip
// and its epilogue's memory accesses are a third of its time.
//   forward    k >= 3: X = Q^2, then Horner's rule in X on the pairs of powers,
//              G - I = sum_i X^i (c_{2i+1} Q + c_{2i+2} X),  c_p = 2 for p <= k, 1 for p = k + 1:
//              1 + floor(k/2) products; k <= 2: Horner's rule in Q, as many products without X
//   backward   P_0 = D = dL/dG,  P_m = D + P_{m-1} T,  Z_0 = D,  Z_m = P_m + T Z_{m-1},  dL/dQ = Z_k + Z_{k-1}
//              with T = Q^T = -Q (see mfma_cnp_lds.hip).  Launch m makes P_m and Z_m = D + P_{m-1} T + T Z_{m-1}, the
//              latter as one contraction over two operand pairs, so that P_m is only ever written as the bf16 operand of the next
//              launch: 3k - 1 products in k launches.  Adding an fp32 P_m in Z_m's epilogue instead saves k products and
//              loses by its traffic (and a launch) except for a few blocks of the first orders.  us per backward,
//              that / this / the two-sided Horner rule on 256 x 256 tiles: k = 3: 16 blocks 102 / 91 / 139,
//              40: 226 / 204 / 203, 48: 272 / 241 / 242, 160: 900 / 808 / 854; k = 5: 16: 147 / 133 / 214, 32: 254 / 242 / 245,
//              48: 400 / 364 / 374, 64: 515 / 465 / 512, 160: 1315 / 1200 / 1346.
// Against 64 bits the recurrences round less than the Horner forms (b = 512, k = 5: 3.8e-4 -> 3.5e-4 of the gradient, 2.67e-4 -> 2.66e-4
// of G - I before its own rounding).
#include "mfma_gemm.h"

namespace poetx {
namespace {

// Tiled products (block sides that do not fit on chip, i.e. b = 512): 128 x 128 tiles, 2 x 2 waves,
// 64 KB of LDS so that two workgroups share a CU; a contraction is only b deep, so the loop
// stops loading after the last tile instead of re-fetching it.
constexpr int CBM = 128, CBN = 128, CBK = 64, CNS = 4;

__global__ void to_bf16_kernel(const float4* __restrict__ in, uint2* __restrict__ out, i64 n4) {
  i64 idx = (i64)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= n4) return;
  float4 v = in[idx];
  uint2 o;
  o.x = mm::pack2_bf16(v.x, v.y);
  o.y = mm::pack2_bf16(v.z, v.w);
  out[idx] = o;
}

// Forward.  FIRST: acc = X; C (in: Q, out: 2Q + 2X), Xb = bf16(X), value v = 2Q + X.  Otherwise v = acc + C.
// Writes whichever outputs are set: Hn (bf16 chain value), G (fp32, + I), E (bf16 pair [nb][2][b][b]: value and its transpose).
template <bool FIRST>
struct EpiFwd {
  float* C;
  uint16_t* Xb;
  int b;
  uint16_t* Hn;
  float* G;
  uint16_t* E;
  __device__ void operator()(int j, int, int row, int col, float4 lo, float4 hi) const {
    const i64 o = ((i64)j * b + row) * b + col;
    const float4 c0 = *reinterpret_cast<const float4*>(C + o), c1 = *reinterpret_cast<const float4*>(C + o + 4);
    const float c[8] = {c0.x, c0.y, c0.z, c0.w, c1.x, c1.y, c1.z, c1.w}, a[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = FIRST ? a[e] + 2.f * c[e] : a[e] + c[e];
    if (FIRST && Xb) {
      *reinterpret_cast<uint4*>(Xb + o) = make_uint4(mm::pack2_bf16(a[0], a[1]), mm::pack2_bf16(a[2], a[3]), mm::pack2_bf16(a[4], a[5]), mm::pack2_bf16(a[6], a[7]));
      *reinterpret_cast<float4*>(C + o) = make_float4(v[0] + a[0], v[1] + a[1], v[2] + a[2], v[3] + a[3]);
      *reinterpret_cast<float4*>(C + o + 4) = make_float4(v[4] + a[4], v[5] + a[5], v[6] + a[6], v[7] + a[7]);
    }
    const uint4 pk = make_uint4(mm::pack2_bf16(v[0], v[1]), mm::pack2_bf16(v[2], v[3]), mm::pack2_bf16(v[4], v[5]), mm::pack2_bf16(v[6], v[7]));
    if (Hn) *reinterpret_cast<uint4*>(Hn + o) = pk;
    if (G) {
      float gv[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) gv[e] = v[e] + (row == col + e ? 1.f : 0.f);
      *reinterpret_cast<float4*>(G + o) = make_float4(gv[0], gv[1], gv[2], gv[3]);
      *reinterpret_cast<float4*>(G + o + 4) = make_float4(gv[4], gv[5], gv[6], gv[7]);
    }
    if (E) {
      const i64 base = (i64)j * 2 * b * b;
      *reinterpret_cast<uint4*>(E + base + (i64)row * b + col) = pk;
#pragma unroll
      for (int e = 0; e < 8; ++e) E[base + (i64)b * b + (i64)(col + e) * b + row] = float_to_bf16_bits(v[e]);
    }
  }
};

// Backward: batches [0, nb) are the first problem of a launch, [nb, 2 nb) the second.  value = acc + add (+ add2), written
// as bf16 and / or fp32 (the fp32 output may take the place of either addend: same element, same thread).
struct EpiAdd {
  struct Side {
    const float* add;
    const float* add2;
    uint16_t* bf;
    float* f;
  } s[2];
  int b, nb;
  __device__ void operator()(int batch, int, int row, int col, float4 lo, float4 hi) const {
    const bool second = batch >= nb;
    const Side& d = s[second ? 1 : 0];
    const i64 o = ((i64)(second ? batch - nb : batch) * b + row) * b + col;
    float4 a0 = *reinterpret_cast<const float4*>(d.add + o), a1 = *reinterpret_cast<const float4*>(d.add + o + 4);
    a0 = make_float4(a0.x + lo.x, a0.y + lo.y, a0.z + lo.z, a0.w + lo.w);
    a1 = make_float4(a1.x + hi.x, a1.y + hi.y, a1.z + hi.z, a1.w + hi.w);
    if (d.add2) {
      const float4 b0 = *reinterpret_cast<const float4*>(d.add2 + o), b1 = *reinterpret_cast<const float4*>(d.add2 + o + 4);
      a0 = make_float4(a0.x + b0.x, a0.y + b0.y, a0.z + b0.z, a0.w + b0.w);
      a1 = make_float4(a1.x + b1.x, a1.y + b1.y, a1.z + b1.z, a1.w + b1.w);
    }
    if (d.bf) *reinterpret_cast<uint4*>(d.bf + o) = make_uint4(mm::pack2_bf16(a0.x, a0.y), mm::pack2_bf16(a0.z, a0.w), mm::pack2_bf16(a1.x, a1.y), mm::pack2_bf16(a1.z, a1.w));
    if (d.f) {
      *reinterpret_cast<float4*>(d.f + o) = a0;
      *reinterpret_cast<float4*>(d.f + o + 4) = a1;
    }
  }
};

// 128 x 128 tiles: 256 x 256 ones have four times the work per workgroup for the same fill and drain, but leave most of the
// chip idle below 128 blocks (build + backward of 16 blocks, k = 5: 327 against 191 us; 64 blocks: 650 against 634).
mm::Args batched_args(int b) {
  mm::Args g{};
  g.tiles_m = b / CBM;
  g.tiles_n = b / CBN;
  return g;
}
template <bool PAIR, class Epi>
void launch_product(const mm::Args& g, Epi epi, int batches, hipStream_t st) {
  mm::launch<CBM, CBN, 2, 2, true, false, false, CNS, PAIR>(g, epi, batches, 1, st);
}
// Blocks worked off together, of those left: what passes from launch to launch (4 MB a block in the backward, rewritten in place by
// the next group) stays largely in the 256 MB memory-side cache; a short remainder joins the last group, as a launch of its own
// costs the same however few its blocks.  All but the last group are a multiple of 8, which keeps the tiles of a block on one
// XCD.  Build + backward at k = 5, us, groups of 32 (last up to 40) / 64 (last up to 80) / all at once:
// 48 blocks 515 / 493 / -, 64: 663 / 634 / -, 80: 858 / 848 / -, 96: 1009 / 995 / 1082, 160: 1709 / 1631 / 1980.
inline int group_size(int left) { return left <= 80 ? left : 64; }
void set_src(mm::Source& s, const uint16_t* A, const uint16_t* B, int b) {
  s.A = A; s.B = B; s.lda = b; s.ldb = b; s.sA = (i64)b * b; s.sB = (i64)b * b; s.ktiles = b / CBK;
}

}  // namespace

bool mfma_cnp_supported(int d, int b) { return (b == 256 || b == 512) && d % b == 0; }

// ws: 3 floats per block element: Q (later 2Q + 2X) in fp32, then bf16(Q), bf16(X) and two chain values.
void mfma_cnp_build(const float* theta, int d, int b, int k, float* G_f32, void* E_bf16, float* ws, hipStream_t st) {
  const int all = d / b;
  if (lds_cnp_supported(d, b)) {   // whole chain in one launch, rows of the block in registers
    lds_cnp_build(theta, all, k, G_f32, E_bf16, ws, st);
    return;
  }
  const i64 bb = (i64)b * b;
  for (int j0 = 0, nb; j0 < all; j0 += nb) {
    nb = group_size(all - j0);
    const i64 total = nb * bb;
    float* C = ws;
    uint16_t* Qb = (uint16_t*)(C + total);
    uint16_t* Xb = Qb + total;
    uint16_t* H[2] = {Xb + total, Xb + 2 * total};
    float* G = G_f32 ? G_f32 + j0 * bb : nullptr;
    uint16_t* E = E_bf16 ? (uint16_t*)E_bf16 + 2 * j0 * bb : nullptr;
    skew_materialize_tiled_launch(theta + j0 * (bb - b) / 2, b, nb, C, Qb, nullptr, st);
    mm::Args g = batched_args(b);
    if (k <= 2) {                    // H = Q Q + 2Q (k = 1: that is it), H Q + 2Q
      set_src(g.s, Qb, Qb, b);
      if (k == 2) {
        launch_product<false>(g, EpiFwd<true>{C, nullptr, b, H[0], nullptr, nullptr}, nb, st);
        set_src(g.s, H[0], Qb, b);
      }
      launch_product<false>(g, EpiFwd<true>{C, nullptr, b, nullptr, G, E}, nb, st);
      continue;
    }
    // the top pair of powers is Q alone for even k, 2Q + X for odd k (then the chain starts in this launch's epilogue)
    const int pairs = k / 2;         // Horner steps in X
    const bool odd = k & 1;
    set_src(g.s, Qb, Qb, b);
    launch_product<false>(g, EpiFwd<true>{C, Xb, b, odd ? H[0] : nullptr, nullptr, nullptr}, nb, st);
    const uint16_t* cur = odd ? H[0] : Qb;
    for (int i = 1; i <= pairs; ++i) {
      const bool last = i == pairs;
      set_src(g.s, Xb, cur, b);
      uint16_t* nxt = H[i & 1];
      launch_product<false>(g, EpiFwd<false>{C, nullptr, b, last ? nullptr : nxt, last ? G : nullptr, last ? E : nullptr}, nb, st);
      cur = nxt;
    }
  }
}

void mfma_cnp_bwd(const SeriesSide* sides, int nsides, int b, int k, int accumulate, float* ws, hipStream_t st) {
  if (lds_cnp_supported(sides[0].d, b)) {   // one launch, left factors in registers
    lds_cnp_bwd(sides, nsides, k, accumulate, ws, st);
    return;
  }
  // blocks of the sides one after the other; their dG must be contiguous in that order
  const int nb0 = sides[0].d / b, nb1 = nsides > 1 ? sides[1].d / b : 0, all = nb0 + nb1;
  const i64 bb = (i64)b * b, L = (bb - b) / 2;
  uint16_t* T_all = (uint16_t*)ws;                       // -Q of all blocks, the rest for a group at a time
  ws += all * bb / 2;
  skew_materialize_tiled_launch(sides[0].theta, b, nb0, nullptr, nullptr, T_all, st);
  if (nb1) skew_materialize_tiled_launch(sides[1].theta, b, nb1, nullptr, nullptr, T_all + nb0 * bb, st);
  for (int j0 = 0, nb; j0 < all; j0 += nb) {
    nb = group_size(all - j0);
    const i64 total = nb * bb;
    const float* D = sides[0].dG + j0 * bb;
    const uint16_t* Tb = T_all + j0 * bb;
    float* Zf = ws;                  // Z_{k-1}, then dL/dQ
    uint16_t* Db = (uint16_t*)(ws + total);
    uint16_t* P[2] = {Db + total, Db + 2 * total};
    uint16_t* Z[2] = {Db + 3 * total, Db + 4 * total};
    hipLaunchKernelGGL(to_bf16_kernel, dim3(ceil_div(total / 4, 256)), dim3(256), 0, st, (const float4*)D, (uint2*)Db, total / 4);
    const uint16_t *p = Db, *z = Db;
    for (int m = 1; m <= k; ++m) {
      const bool last = m == k;
      mm::Args g = batched_args(b);
      set_src(g.s, p, Tb, b);        // Z_m
      set_src(g.s2, Tb, z, b);
      EpiAdd epi{};
      epi.b = b;
      epi.nb = nb;
      epi.s[0] = {D, !last ? nullptr : k > 1 ? Zf : D, last ? nullptr : Z[m & 1], m >= k - 1 ? Zf : nullptr};
      if (!last) {                   // P_m
        g.alt_from = nb;
        set_src(g.alt, p, Tb, b);
        epi.s[1] = {D, nullptr, P[m & 1], nullptr};
      }
      launch_product<true>(g, epi, last ? nb : 2 * nb, st);
      p = P[m & 1];
      z = Z[m & 1];
    }
    const int n0 = nb0 - j0 < 0 ? 0 : nb0 - j0 < nb ? nb0 - j0 : nb, j1 = j0 + n0 - nb0;       // of the group: blocks of the first side, first block of the second
    skew_project_sides_launch(Zf, b, n0, sides[0].dtheta + j0 * L, nb - n0, nb > n0 ? sides[1].dtheta + j1 * L : nullptr, accumulate, st);
  }
}

}  // namespace poetx
