// Local stiffness action w = D^T G D u (paper section 4.2.1) with the six
// tensor contractions on the matrix cores: BF16 inputs u and G, FP32
// accumulation, FP32 output.
//
// The derivative matrix cannot simply be rounded to BF16: its rounding error
// does not vanish on smooth inputs (D 1 != 0, D x != 1), which the
// refinement around the operator cannot undo.  It is split instead,
// D = D_hi + D_lo with D_hi = bf16(D) and D_lo = bf16(D - D_hi) (a two-term
// BF16 expansion, relative error ~2^-16), and every contraction runs as two
// accumulating MFMAs.  SPLIT = false keeps only D_hi (the inaccurate
// variant, kept for measurement).
//
// One wave per element, the element padded to 8^3 nodes (n1 <= 8; padded
// entries of u and D are zero), four waves per workgroup, each with its own
// LDS region: the phases of an element are ordered by wave-level barriers,
// so the waves of a workgroup do not wait for each other.  MFMA tile
// 16x16x16 (v_mfma_f32_16x16x16_bf16): lane l = 16 g + r holds A[r][4g + q],
// B[4g + q][r] and C[4g + q][r], q = 0..3.  A length-8 contraction uses a
// block-diagonal operand diag(D, D) so that one MFMA contracts two 8-blocks:
//   t (over k):  C[(b,k)][c']   = sum_m D[k][m] u[m][cb + 16 b + c']
//   r (over i):  C[rho'][(b,i)] = sum_m u[rb + 16 b + rho'][m] D[i][m]
//   s (over j):  C[(b,j)][(h,i)] = sum_m D[j][m] u[kb + 2 b + h][m][i]
// with c = (j,i) and rho = (k,j); two MFMAs (cb, rb, kb) cover the element.
// The transposed contractions use D^T the same way and accumulate w through
// the C operand (r, then s, then t), staged in LDS in [k][j][i] order.  The
// metric step between them (fluxes = G grad u) is FP32 on the VALU, one lane
// per (i,j) column, and the fluxes are rounded to BF16 for the MFMAs.  With a
// mass term the lumped H o u (H = alpha(X) B in BF16) is added in FP32 as the
// result leaves LDS.
#include <algorithm>

#include "ax_tile.h"

namespace sem {

typedef short m16x4 __attribute__((ext_vector_type(4)));
typedef float mf32x4 __attribute__((ext_vector_type(4)));
// (the output need only be aligned to its element)
typedef float mf32x4_u __attribute__((ext_vector_type(4), aligned(4)));

constexpr int MW = 4;  // waves (elements) per workgroup
// elements per launch, a wave each: a launch holds fewer than 2^32 threads
constexpr int64_t MFMA_PIECE = (int64_t)1 << 25;

struct alignas(16) MfmaLds {
  uint16_t u[512];                  // u (BF16), or the high term of its split
  float gr[512], gs[512], gt[512];  // gradients; gr is reused for w
  uint16_t fr[512], fs[512], ft[512];
};
// with the low term of a split input: ul = bf16(u - bf16(u))
struct alignas(16) MfmaLdsSplit : MfmaLds {
  uint16_t ul[512];
};

__device__ inline m16x4 lds4_strided(const uint16_t *p, int stride) {
  m16x4 v;
  v[0] = (short)p[0];
  v[1] = (short)p[stride];
  v[2] = (short)p[2 * stride];
  v[3] = (short)p[3 * stride];
  return v;
}

__device__ inline mf32x4 mfma(m16x4 a, m16x4 b, mf32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

// Operands of the derivative matrix held by lane l (constant per kernel):
//   fwd[q] = D[r % 8][4 (g % 2) + q], bwd[q] = D[4 (g % 2) + q][r % 8],
// zero off the diagonal blocks (r / 8 != g / 2) and outside n1.
template <int N1>
__device__ inline void d_operands(int l, const uint16_t *__restrict__ Dhi_,
                                  const uint16_t *__restrict__ Dlo_, m16x4 &fh,
                                  m16x4 &fl, m16x4 &bh, m16x4 &bl) {
  const gp<const uint16_t> Dhi = (gp<const uint16_t>)Dhi_;
  const gp<const uint16_t> Dlo = (gp<const uint16_t>)Dlo_;
  const int r = l & 15, g = l >> 4;
  const bool blk = (r >> 3) == (g >> 1);
  const int a = r & 7;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int m = 4 * (g & 1) + q;
    const bool okf = blk && a < N1 && m < N1;
    fh[q] = okf ? (short)Dhi[a * N1 + m] : (short)0;
    fl[q] = okf ? (short)Dlo[a * N1 + m] : (short)0;
    bh[q] = okf ? (short)Dhi[m * N1 + a] : (short)0;
    bl[q] = okf ? (short)Dlo[m * N1 + a] : (short)0;
  }
}

// One element per wave.  The caller has placed the element's u (BF16,
// padded [k][j][i] order, zeros outside n1) in L.u -- with ULO, an FP32 u
// as the two-term split u = L.u + L.ul -- and holds in gq the six BF16
// factors of the lane's column (i, j) = (l % 8, l / 8) for k < 8 (zero
// outside the element).  On return L.gr holds w in [k][j][i] order.  With
// ULO each gradient contraction accumulates D_hi u_hi, D_lo u_hi and
// D_hi u_lo (the D_lo u_lo term is below the FP32 accumulation's rounding).
template <int N1, bool SPLIT, bool ULO = false, class Lds = MfmaLds>
__device__ inline void mfma_element(int l, Lds &L, const uint16_t (&gq)[6][8],
                                    m16x4 fh, m16x4 fl, m16x4 bh, m16x4 bl) {
  const int r = l & 15, g = l >> 4;
  const mf32x4 zero = {0.f, 0.f, 0.f, 0.f};
  // ---- gradient: three contractions ----
#pragma unroll
  for (int h2 = 0; h2 < 2; ++h2) {
    {  // t: B from u[m][c], m = 4 (g % 2) + q, c = 32 h2 + 16 (g / 2) + r
      const int c = 32 * h2 + 16 * (g >> 1) + r, m0 = 4 * (g & 1);
      const m16x4 b = lds4_strided(&L.u[m0 * 64 + c], 64);
      mf32x4 acc = mfma(fh, b, zero);
      if (SPLIT) acc = mfma(fl, b, acc);
      if constexpr (ULO) acc = mfma(fh, lds4_strided(&L.ul[m0 * 64 + c], 64), acc);
#pragma unroll
      for (int q = 0; q < 4; ++q) L.gt[(m0 + q) * 64 + c] = acc[q];
    }
    {  // r: A from u[rho][m], rho = 32 h2 + 16 (g / 2) + r
      const int rho = 32 * h2 + 16 * (g >> 1) + r, m0 = 4 * (g & 1);
      const m16x4 a = *reinterpret_cast<const m16x4 *>(&L.u[rho * 8 + m0]);
      mf32x4 acc = mfma(a, fh, zero);
      if (SPLIT) acc = mfma(a, fl, acc);
      if constexpr (ULO)
        acc = mfma(*reinterpret_cast<const m16x4 *>(&L.ul[rho * 8 + m0]), fh, acc);
      const int i = r & 7, rho0 = 32 * h2 + 16 * (r >> 3) + 4 * g;
#pragma unroll
      for (int q = 0; q < 4; ++q) L.gr[(rho0 + q) * 8 + i] = acc[q];
    }
    {  // s: B from u[k][m][i], k = 4 h2 + 2 (g / 2) + r / 8
      const int k = 4 * h2 + 2 * (g >> 1) + (r >> 3), i = r & 7, m0 = 4 * (g & 1);
      const m16x4 b = lds4_strided(&L.u[k * 64 + m0 * 8 + i], 8);
      mf32x4 acc = mfma(fh, b, zero);
      if (SPLIT) acc = mfma(fl, b, acc);
      if constexpr (ULO) acc = mfma(fh, lds4_strided(&L.ul[k * 64 + m0 * 8 + i], 8), acc);
#pragma unroll
      for (int q = 0; q < 4; ++q) L.gs[k * 64 + (m0 + q) * 8 + i] = acc[q];
    }
  }
  wave_lds_sync();
  // ---- metric step on the lane's column (FP32) ----
  {
    const int i = l & 7, j = l >> 3;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int p = k * 64 + j * 8 + i;
      const float ur = L.gr[p], us = L.gs[p], ut = L.gt[p];
      const float g0 = bf16_to_f32(gq[0][k]), g1 = bf16_to_f32(gq[1][k]),
                  g2 = bf16_to_f32(gq[2][k]), g3 = bf16_to_f32(gq[3][k]),
                  g4 = bf16_to_f32(gq[4][k]), g5 = bf16_to_f32(gq[5][k]);
      L.fr[p] = f32_to_bf16(g0 * ur + g1 * us + g2 * ut);
      L.fs[p] = f32_to_bf16(g1 * ur + g3 * us + g4 * ut);
      L.ft[p] = f32_to_bf16(g2 * ur + g4 * us + g5 * ut);
    }
  }
  wave_lds_sync();
  // ---- divergence: w = D_r^T f_r + D_s^T f_s + D_t^T f_t into L.gr ----
#pragma unroll
  for (int h2 = 0; h2 < 2; ++h2) {  // r: A from f_r[rho][m], B = D^T blocks
    const int rho = 32 * h2 + 16 * (g >> 1) + r, m0 = 4 * (g & 1);
    const m16x4 a = *reinterpret_cast<const m16x4 *>(&L.fr[rho * 8 + m0]);
    mf32x4 acc = mfma(a, bh, zero);
    if (SPLIT) acc = mfma(a, bl, acc);
    const int i = r & 7, rho0 = 32 * h2 + 16 * (r >> 3) + 4 * g;
#pragma unroll
    for (int q = 0; q < 4; ++q) L.gr[(rho0 + q) * 8 + i] = acc[q];
  }
  wave_lds_sync();
#pragma unroll
  for (int h2 = 0; h2 < 2; ++h2) {  // s: A = diag(D^T), B from f_s[k][m][i]
    const int k = 4 * h2 + 2 * (g >> 1) + (r >> 3), i = r & 7, m0 = 4 * (g & 1);
    const m16x4 b = lds4_strided(&L.fs[k * 64 + m0 * 8 + i], 8);
    mf32x4 acc;
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[q] = L.gr[k * 64 + (m0 + q) * 8 + i];
    acc = mfma(bh, b, acc);
    if (SPLIT) acc = mfma(bl, b, acc);
#pragma unroll
    for (int q = 0; q < 4; ++q) L.gr[k * 64 + (m0 + q) * 8 + i] = acc[q];
  }
  wave_lds_sync();
#pragma unroll
  for (int h2 = 0; h2 < 2; ++h2) {  // t: A = diag(D^T), B from f_t[m][c]
    const int c = 32 * h2 + 16 * (g >> 1) + r, m0 = 4 * (g & 1);
    const m16x4 b = lds4_strided(&L.ft[m0 * 64 + c], 64);
    mf32x4 acc;
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[q] = L.gr[(m0 + q) * 64 + c];
    acc = mfma(bh, b, acc);
    if (SPLIT) acc = mfma(bl, b, acc);
#pragma unroll
    for (int q = 0; q < 4; ++q) L.gr[(m0 + q) * 64 + c] = acc[q];
  }
  wave_lds_sync();
}

// the six BF16 factors of column (i, j) of element e: the column-contiguous
// layout [E][6][64][8] at n1 = 8, [E][6][n1^3] otherwise.  nt (n1 = 8): with
// the streaming hint, for operators beyond the last-level cache (OpShape)
template <int N1>
__device__ inline void load_factors(int l, bool act, int64_t e, bool nt,
                                    const uint16_t *__restrict__ G_,
                                    uint16_t (&gq)[6][8]) {
  constexpr int NP = N1 * N1, N3 = NP * N1;
  const gp<const uint16_t> G = (gp<const uint16_t>)G_;
  const int i = l & 7, j = l >> 3;
  if constexpr (N1 == 8) {
#pragma unroll
    for (int q = 0; q < 6; ++q) {
      u32x4 v = {0u, 0u, 0u, 0u};
      const gp<const u32x4> row = (gp<const u32x4>)(G + e * 6 * N3 + q * N3 + 8 * l);
      if (act) v = nt ? __builtin_nontemporal_load(row) : *row;
      const uint32_t wv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int h = 0; h < 4; ++h) {
        gq[q][2 * h] = (uint16_t)(wv[h] & 0xffffu);
        gq[q][2 * h + 1] = (uint16_t)(wv[h] >> 16);
      }
    }
  } else {
    const bool col = act && i < N1 && j < N1;
#pragma unroll
    for (int q = 0; q < 6; ++q)
#pragma unroll
      for (int k = 0; k < 8; ++k)
        gq[q][k] = (col && k < N1)
                       ? G[e * 6 * N3 + q * N3 + k * NP + j * N1 + i]
                       : (uint16_t)0;
  }
}

// ---------------------------------------------------------------------------
// n1 = 9 (N = 8): the element does not fit the 8-block form.  Every
// contraction runs on 16-padded operands instead: the derivative operand is
// D (or D^T) padded to 16 x 16 with zeros, the node operand is read from the
// element's natural [k][j][i] layout in LDS with every index beyond 8
// predicated to zero, and one 16x16x16 MFMA contracts a whole length-9
// line:
//   t (over k):  C[k'][c]    = sum_m D[k'][m] u[m][c],  c = (j, i) in 6
//                tiles of 16 of the 81 columns
//   r (over i):  C[rho][i']  = sum_m u[rho][m] D[i'][m], rho = (k, j) in 6
//                tiles of 16 of the 81 rows
//   s (over j):  C[j'][i]    = sum_m D[j'][m] u[k][m][i], one MFMA per k
// (21 MFMAs per derivative term and direction set, against 6 with the
// block-diagonal 8-form; the matrix cores are far from busy either way).
// The transposed contractions use D^T the same way and accumulate w through
// the C operand (r, then s, then t).  The metric step is FP32 on the VALU,
// lane l taking the columns l and l + 64 (< 81).
// ---------------------------------------------------------------------------
constexpr int MW9 = 2;  // waves (elements) per workgroup at n1 = 9
constexpr int E9 = 729;

struct alignas(16) MfmaLds9 {
  uint16_t u[E9];
  uint16_t ul[E9];                  // low term of a split input (solver)
  float gr[E9], gs[E9], gt[E9];     // gradients; gr is reused for w
  uint16_t fr[E9], fs[E9], ft[E9];
};

// D[r][4g + q] (fwd) and D[4g + q][r] (bwd), zero outside 9 x 9
__device__ inline void d_operands9(int l, const uint16_t *__restrict__ Dhi_,
                                   const uint16_t *__restrict__ Dlo_, m16x4 &fh,
                                   m16x4 &fl, m16x4 &bh, m16x4 &bl) {
  const gp<const uint16_t> Dhi = (gp<const uint16_t>)Dhi_;
  const gp<const uint16_t> Dlo = (gp<const uint16_t>)Dlo_;
  const int r = l & 15, g = l >> 4;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int m = 4 * g + q;
    const bool ok = r < 9 && m < 9;
    fh[q] = ok ? (short)Dhi[r * 9 + m] : (short)0;
    fl[q] = ok ? (short)Dlo[r * 9 + m] : (short)0;
    bh[q] = ok ? (short)Dhi[m * 9 + r] : (short)0;
    bl[q] = ok ? (short)Dlo[m * 9 + r] : (short)0;
  }
}

// four BF16 values p[off(q)], q = 0..3, zero where ok(q) fails
template <class F, class O>
__device__ inline m16x4 lds4_pred(const uint16_t *p, F off, O ok) {
  m16x4 v;
#pragma unroll
  for (int q = 0; q < 4; ++q) v[q] = ok(q) ? (short)p[off(q)] : (short)0;
  return v;
}

// One element per wave, u (BF16, [k][j][i], with ULO the FP32 split u =
// L.u + L.ul) in LDS; gq holds the BF16 factors of the lane's columns l and
// l + 64 for k = 0..8.  On return L.gr holds w in [k][j][i] order.
template <bool SPLIT, bool ULO>
__device__ inline void mfma_element9(int l, MfmaLds9 &L, const uint16_t (&gq)[2][6][9],
                                     m16x4 fh, m16x4 fl, m16x4 bh, m16x4 bl) {
  const int r = l & 15, g = l >> 4;
  const mf32x4 zero = {0.f, 0.f, 0.f, 0.f};
  // ---- gradient ----
#pragma unroll
  for (int t = 0; t < 6; ++t) {  // t: columns c = 16 t + r
    const int c = 16 * t + r;
    auto off = [&](int q) { return (4 * g + q) * 81 + c; };
    auto ok = [&](int q) { return 4 * g + q < 9 && c < 81; };
    const m16x4 b = lds4_pred(L.u, off, ok);
    mf32x4 acc = mfma(fh, b, zero);
    if (SPLIT) acc = mfma(fl, b, acc);
    if constexpr (ULO) acc = mfma(fh, lds4_pred(L.ul, off, ok), acc);
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (4 * g + q < 9 && c < 81) L.gt[(4 * g + q) * 81 + c] = acc[q];
  }
#pragma unroll
  for (int t = 0; t < 6; ++t) {  // r: rows rho = 16 t + r of u[rho][m]
    const int rho = 16 * t + r;
    auto off = [&](int q) { return rho * 9 + 4 * g + q; };
    auto ok = [&](int q) { return rho < 81 && 4 * g + q < 9; };
    const m16x4 a = lds4_pred(L.u, off, ok);
    mf32x4 acc = mfma(a, fh, zero);
    if (SPLIT) acc = mfma(a, fl, acc);
    if constexpr (ULO) acc = mfma(lds4_pred(L.ul, off, ok), fh, acc);
    // C[rho'][i'] with rho' = 16 t + 4 g + q, i' = r
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int rr = 16 * t + 4 * g + q;
      if (rr < 81 && r < 9) L.gr[rr * 9 + r] = acc[q];
    }
  }
#pragma unroll
  for (int k = 0; k < 9; ++k) {  // s: B[m][i] = u[k][m][i]
    auto off = [&](int q) { return k * 81 + (4 * g + q) * 9 + r; };
    auto ok = [&](int q) { return 4 * g + q < 9 && r < 9; };
    const m16x4 b = lds4_pred(L.u, off, ok);
    mf32x4 acc = mfma(fh, b, zero);
    if (SPLIT) acc = mfma(fl, b, acc);
    if constexpr (ULO) acc = mfma(fh, lds4_pred(L.ul, off, ok), acc);
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (4 * g + q < 9 && r < 9) L.gs[k * 81 + (4 * g + q) * 9 + r] = acc[q];
  }
  wave_lds_sync();
  // ---- metric step on the lane's columns (FP32) ----
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int c = l + 64 * h;
    if (c < 81) {
#pragma unroll
      for (int k = 0; k < 9; ++k) {
        const int p = k * 81 + c;
        const float ur = L.gr[p], us = L.gs[p], ut = L.gt[p];
        const float g0 = bf16_to_f32(gq[h][0][k]), g1 = bf16_to_f32(gq[h][1][k]),
                    g2 = bf16_to_f32(gq[h][2][k]), g3 = bf16_to_f32(gq[h][3][k]),
                    g4 = bf16_to_f32(gq[h][4][k]), g5 = bf16_to_f32(gq[h][5][k]);
        L.fr[p] = f32_to_bf16(g0 * ur + g1 * us + g2 * ut);
        L.fs[p] = f32_to_bf16(g1 * ur + g3 * us + g4 * ut);
        L.ft[p] = f32_to_bf16(g2 * ur + g4 * us + g5 * ut);
      }
    }
  }
  wave_lds_sync();
  // ---- divergence into L.gr ----
#pragma unroll
  for (int t = 0; t < 6; ++t) {  // r: A = f_r[rho][m], B[m][i] = D[m][i]
    const int rho = 16 * t + r;
    auto off = [&](int q) { return rho * 9 + 4 * g + q; };
    auto ok = [&](int q) { return rho < 81 && 4 * g + q < 9; };
    const m16x4 a = lds4_pred(L.fr, off, ok);
    mf32x4 acc = mfma(a, bh, zero);
    if (SPLIT) acc = mfma(a, bl, acc);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int rr = 16 * t + 4 * g + q;
      if (rr < 81 && r < 9) L.gr[rr * 9 + r] = acc[q];
    }
  }
  wave_lds_sync();
#pragma unroll
  for (int k = 0; k < 9; ++k) {  // s: A[j][m] = D[m][j], B[m][i] = f_s[k][m][i]
    auto off = [&](int q) { return k * 81 + (4 * g + q) * 9 + r; };
    auto ok = [&](int q) { return 4 * g + q < 9 && r < 9; };
    const m16x4 b = lds4_pred(L.fs, off, ok);
    mf32x4 acc;
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[q] = ok(q) ? L.gr[off(q)] : 0.f;
    acc = mfma(bh, b, acc);
    if (SPLIT) acc = mfma(bl, b, acc);
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (ok(q)) L.gr[off(q)] = acc[q];
  }
  wave_lds_sync();
#pragma unroll
  for (int t = 0; t < 6; ++t) {  // t: A[k][m] = D[m][k], B[m][c] = f_t[m][c]
    const int c = 16 * t + r;
    auto off = [&](int q) { return (4 * g + q) * 81 + c; };
    auto ok = [&](int q) { return 4 * g + q < 9 && c < 81; };
    const m16x4 b = lds4_pred(L.ft, off, ok);
    mf32x4 acc;
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[q] = ok(q) ? L.gr[off(q)] : 0.f;
    acc = mfma(bh, b, acc);
    if (SPLIT) acc = mfma(bl, b, acc);
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (ok(q)) L.gr[off(q)] = acc[q];
  }
  wave_lds_sync();
}

// the BF16 factors of columns l and l + 64 of element e ([E][6][729])
__device__ inline void load_factors9(int l, bool act, int64_t e,
                                     const uint16_t *__restrict__ G_,
                                     uint16_t (&gq)[2][6][9]) {
  const gp<const uint16_t> G = (gp<const uint16_t>)G_;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int c = l + 64 * h;
    const bool col = act && c < 81;
#pragma unroll
    for (int q = 0; q < 6; ++q)
#pragma unroll
      for (int k = 0; k < 9; ++k)
        gq[h][q][k] = col ? G[e * 6 * E9 + q * E9 + k * 81 + c] : (uint16_t)0;
  }
}

template <bool SPLIT>
__global__ void __launch_bounds__(64 * MW9)
    k_ax_mfma9(int64_t E, const uint16_t *__restrict__ Dhi,
               const uint16_t *__restrict__ Dlo, const uint16_t *__restrict__ G,
               const uint16_t *__restrict__ H, const uint16_t *__restrict__ u,
               float *__restrict__ w) {
  __shared__ MfmaLds9 lds[MW9];
  const int wv = threadIdx.x >> 6, l = threadIdx.x & 63;
  const int64_t e = (int64_t)blockIdx.x * MW9 + wv;
  const bool act = e < E;
  MfmaLds9 &L = lds[wv];
  m16x4 fh, fl, bh, bl;
  d_operands9(l, Dhi, Dlo, fh, fl, bh, bl);
  uint16_t gq[2][6][9];
  load_factors9(l, act, e, G, gq);
  for (int p = l; p < E9; p += 64) L.u[p] = act ? u[e * E9 + p] : (uint16_t)0;
  wave_lds_sync();
  mfma_element9<SPLIT, false>(l, L, gq, fh, fl, bh, bl);
  if (!act) return;  // no barrier follows
  for (int p = l; p < E9; p += 64) {
    float v = L.gr[p];
    if (H != nullptr) v += bf16_to_f32(H[e * E9 + p]) * bf16_to_f32(L.u[p]);
    w[e * E9 + p] = v;
  }
}

// ---------------------------------------------------------------------------
// standalone operator: BF16 E-vector in, FP32 E-vector out
// ---------------------------------------------------------------------------
template <int N1, bool SPLIT>
__global__ void __launch_bounds__(64 * MW)
    k_ax_mfma(int64_t E, const uint16_t *__restrict__ Dhi,
              const uint16_t *__restrict__ Dlo, const uint16_t *__restrict__ G,
              const uint16_t *__restrict__ H, const uint16_t *__restrict__ u,
              float *__restrict__ w, int nt) {
  constexpr int NP = N1 * N1, N3 = NP * N1;
  __shared__ MfmaLds lds[MW];
  const int wv = threadIdx.x >> 6, l = threadIdx.x & 63;
  const int64_t e = (int64_t)blockIdx.x * MW + wv;
  const bool act = e < E;
  MfmaLds &L = lds[wv];
  m16x4 fh, fl, bh, bl;
  d_operands<N1>(l, Dhi, Dlo, fh, fl, bh, bl);
  uint16_t gq[6][8];
  load_factors<N1>(l, act, e, nt != 0, G, gq);
  if constexpr (N1 == 8) {
    u32x4 v = {0u, 0u, 0u, 0u};
    if (act) v = *reinterpret_cast<const u32x4 *>(u + e * N3 + 8 * l);
    *reinterpret_cast<u32x4 *>(&L.u[8 * l]) = v;
  } else {
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const int p = l + 64 * t, i = p & 7, j = (p >> 3) & 7, k = p >> 6;
      L.u[p] = (act && i < N1 && j < N1 && k < N1) ? u[e * N3 + k * NP + j * N1 + i]
                                                   : (uint16_t)0;
    }
  }
  wave_lds_sync();
  mfma_element<N1, SPLIT>(l, L, gq, fh, fl, bh, bl);
  if (!act) return;  // no barrier follows
  if constexpr (N1 == 8) {
    const float *src = &L.gr[8 * l];
    float hv[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (H != nullptr) {  // uniform
      const u32x4 v =
          __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(H + e * N3 + 8 * l));
      const uint32_t wv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int h = 0; h < 4; ++h) {
        hv[2 * h] = bf16_to_f32((uint16_t)(wv[h] & 0xffffu)) * bf16_to_f32(L.u[8 * l + 2 * h]);
        hv[2 * h + 1] =
            bf16_to_f32((uint16_t)(wv[h] >> 16)) * bf16_to_f32(L.u[8 * l + 2 * h + 1]);
      }
    }
    // 32 consecutive bytes per lane in two stores
    mf32x4_u *dst = reinterpret_cast<mf32x4_u *>(w + e * N3 + 8 * l);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const mf32x4_u v = {src[4 * h] + hv[4 * h], src[4 * h + 1] + hv[4 * h + 1],
                        src[4 * h + 2] + hv[4 * h + 2], src[4 * h + 3] + hv[4 * h + 3]};
      if (nt)
        __builtin_nontemporal_store(v, dst + h);
      else
        dst[h] = v;
    }
  } else {
    for (int p = l; p < N3; p += 64) {
      const int i = p % N1, j = (p / N1) % N1, k = p / NP;
      const int q = k * 64 + j * 8 + i;
      float v = L.gr[q];
      if (H != nullptr) v += bf16_to_f32(H[e * N3 + p]) * bf16_to_f32(L.u[q]);
      w[e * N3 + p] = v;
    }
  }
}

template <bool SPLIT>
static void launch_ax_mfma_s(int N, int64_t E, const uint16_t *Dhi,
                             const uint16_t *Dlo, const uint16_t *G,
                             const uint16_t *H, const uint16_t *u, float *w, int nt,
                             hipStream_t s) {
  const int64_t blocks = (E + MW - 1) / MW;
  if (blocks == 0) return;
  const dim3 grid((unsigned)blocks), block(64 * MW);
  switch (N) {
#define SEM_AXM(NN)                                                          \
  case NN:                                                                   \
    hipLaunchKernelGGL((k_ax_mfma<NN + 1, SPLIT>), grid, block, 0, s, E, Dhi, \
                       Dlo, G, H, u, w, nt);                                 \
    break;
    SEM_AXM(1)
    SEM_AXM(2)
    SEM_AXM(3)
    SEM_AXM(4)
    SEM_AXM(5)
    SEM_AXM(6)
    SEM_AXM(7)
#undef SEM_AXM
    case 8:
      hipLaunchKernelGGL((k_ax_mfma9<SPLIT>), dim3((unsigned)((E + MW9 - 1) / MW9)),
                         dim3(64 * MW9), 0, s, E, Dhi, Dlo, G, H, u, w);
      break;
    default:
      fail(SEM_ERR_ARG, "sem_ax: the matrix-core operator needs N in 1..8");
  }
}

void launch_ax_mfma(int N, bool split, int64_t E, const uint16_t *Dhi,
                    const uint16_t *Dlo, const uint16_t *G, const uint16_t *H,
                    const uint16_t *u, float *w, hipStream_t s) {
  const int64_t N3 = (int64_t)(N + 1) * (N + 1) * (N + 1);
  const int nt = ax_regime(E * N3, 18) == AX_STREAM;
  for (int64_t e = 0; e < E; e += MFMA_PIECE) {
    const int64_t n = std::min(E - e, MFMA_PIECE);
    auto go = split ? launch_ax_mfma_s<true> : launch_ax_mfma_s<false>;
    go(N, n, Dhi, Dlo, G + 6 * e * N3, H ? H + e * N3 : nullptr, u + e * N3, w + e * N3, nt, s);
    SEM_HIP(hipGetLastError());
  }
}

// ---------------------------------------------------------------------------
// batched operator inside the solvers: FP32 unique-node input gathered
// through the box numbering and split into two BF16 terms (u_hi = bf16(u),
// u_lo = bf16(u - u_hi)), FP32 E-vector output; items are tiles of a single
// order (n1 = N1s), MW elements per workgroup pass.  Rounding the input to
// BF16 alone leaves an input error that refinement cannot remove at scale:
// A (I + Delta) p with |Delta| ~ 2^-9 amplifies rough components by the
// operator's spread of eigenvalues, and the refinement's contraction grew
// with the mesh (0.36 per step at 32^3 elements, N = 7).
// ---------------------------------------------------------------------------
// The solvers apply this operator to the search direction only: its gathered
// input z (mode 3), or p' = z + beta p (cg_dir.h), which is then stored.
struct DirMfma {
  gp<const float> z, p;
  gp<float> pnew;  // null in mode 3
  float beta;
  bool first;      // the direction is z
};

// beta and first of the direction; true when the solve has ended
__device__ inline bool dir_mfma(CgState *st, int mode, const double *part, int stride, int beg,
                                int end, bool writer, DirMfma &dir) {
  const DirScalars s = dir_scalars(st);
  dir.beta = 0.f;
  dir.first = true;
  if (mode == 3) return s.done != 0;
  DirStep ds;
  if (mode == 2) {
    DirParts<true> parts;
    parts.load(part, stride, beg, end);
    ds = dir_step<true>(st, s, parts, writer);
  } else {
    ds = dir_step<false>(st, s, DirParts<false>(), writer);
  }
  dir.beta = (float)ds.beta;
  dir.first = ds.first;
  return ds.stop;
}

// the NT nodes of one lane, node(t, i, j, k) giving each one's place in the
// element (false: no node): p' into v (0 where there is none), stored by the
// element that owns the node
template <int NT, class F>
__device__ inline void gather_dir(const Box &box, const DirMfma &d, bool act, int64_t e,
                                  F node, float (&v)[NT]) {
  ElemXYZ c3 = {0u, 0u, 0u};
  if (act) c3 = box_elem(box, (uint32_t)e);
  int64_t g[NT];
  float po[NT];
  bool own[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    uint32_t i, j, k;
    const bool in = node(t, i, j, k) && act;
    const uint32_t gx = wrap_coord(c3.x * (uint32_t)box.N + i, box.Gx);
    const uint32_t gy = wrap_coord(c3.y * (uint32_t)box.N + j, box.Gy);
    const uint32_t gz = wrap_coord(c3.z * (uint32_t)box.N + k, box.Gz);
    g[t] = (int64_t)gx + (int64_t)box.Gx * ((int64_t)gy + (int64_t)box.Gy * gz);
    v[t] = in ? d.z[g[t]] : 0.f;
    po[t] = in && d.pnew != nullptr ? d.p[g[t]] : 0.f;
    own[t] = in && d.pnew != nullptr && owns_coord(i, c3.x, gx) && owns_coord(j, c3.y, gy) &&
             owns_coord(k, c3.z, gz);
  }
#pragma unroll
  for (int t = 0; t < NT; ++t)
    if (!d.first) v[t] = axpy1(d.beta, po[t], v[t]);
#pragma unroll
  for (int t = 0; t < NT; ++t)
    if (own[t]) d.pnew[g[t]] = v[t];
}

// One element of the solvers' operator (gathered FP32 direction, split into
// two BF16 terms; FP32 output), and the element energy p'_e^T w_e in FP64:
// each lane's column of p' times the stored w in ascending k, then the lanes
// by a fixed butterfly.  Every wave of the workgroup calls it (act = false:
// no loads or stores).
template <int N1, bool SPLIT>
__device__ inline void solve_elem_mfma(int l, MfmaLdsSplit &L, int64_t e, bool act, bool nt,
                                       const Box &box, const DirMfma &dir, gp<float> w,
                                       const uint16_t *G, gp<const uint16_t> H,
                                       m16x4 fh, m16x4 fl, m16x4 bh, m16x4 bl,
                                       gp<double> edot) {
  constexpr int NP = N1 * N1, N3 = NP * N1;
  uint16_t gq[6][8];
  load_factors<N1>(l, act, e, nt, G, gq);
  float pv[8];  // the lane's column (i, j) = (l % 8, l / 8) of p', k = t
  gather_dir(
      box, dir, act, e,
      [&](int t, uint32_t &i, uint32_t &j, uint32_t &k) {
        i = l & 7, j = l >> 3, k = t;
        return i < N1 && j < N1 && k < N1;
      },
      pv);
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    const int p = l + 64 * t;
    const float v = pv[t];
    const uint16_t hi = f32_to_bf16(v);
    L.u[p] = hi;
    L.ul[p] = f32_to_bf16(v - bf16_to_f32(hi));
  }
  wave_lds_sync();
  mfma_element<N1, SPLIT, true, MfmaLdsSplit>(l, L, gq, fh, fl, bh, bl);
  // w at node (i, j, k) of the element, as stored (mass term added)
  auto wval = [&](int i, int j, int k) {
    const int q = k * 64 + j * 8 + i;
    float v = L.gr[q];
    if (H != nullptr)
      v += bf16_to_f32(H[e * N3 + k * NP + j * N1 + i]) *
           (bf16_to_f32(L.u[q]) + bf16_to_f32(L.ul[q]));
    return v;
  };
  if (act) {
    for (int p = l; p < N3; p += 64) w[e * N3 + p] = wval(p % N1, (p / N1) % N1, p / NP);
  }
  const int i = l & 7, j = l >> 3;
  double cd = 0.0;
  if (act && i < N1 && j < N1) {  // (wval reads H at the element)
#pragma unroll
    for (int t = 0; t < N1; ++t) cd += (double)pv[t] * (double)wval(i, j, t);
  }
  cd = wave_sum(cd);
  if (act && l == 0) edot[e] = cd;
}

// the direction of a batch's item; true when the item has nothing to do (the
// solve has ended; its first tile has passed that on)
__device__ inline bool batch_dir_mfma(const BatchSolve &sd, CgState *st, const BaxDir &bd,
                                      const AxItem &it, DirMfma &dir) {
  const bool first_tile = it.elem0 == 0;
  if (st[it.solve].done != 0 && !first_tile) return true;  // (mode 3: dir_mfma)
  const bool writer = first_tile && threadIdx.x == 0;
  const int beg = bd.vbeg[it.solve], end = bd.vbeg[it.solve + 1];
  dir.z = (gp<const float>)sd.v32[bd.mode == 3 ? VP : VZ];
  dir.p = (gp<const float>)sd.v32[bd.par ? VW : VP];
  dir.pnew = bd.mode == 3 ? (gp<float>)nullptr : (gp<float>)sd.v32[bd.par ? VP : VW];
  return dir_mfma(st + it.solve, bd.mode, bd.part, bd.stride, beg, end, writer, dir);
}

// (three waves per SIMD are what the workgroups' LDS allows: without the hint
// N = 6 took the registers of two)
template <int N1, bool SPLIT>
__global__ void __launch_bounds__(64 * MW) __attribute__((amdgpu_waves_per_eu(3)))
    k_bax_mfma(const BatchSolve *__restrict__ sds, CgState *st,
               const AxItem *__restrict__ items, int nitems, int epb, BaxDir bd) {
  __shared__ MfmaLdsSplit lds[MW];
  const int wv = threadIdx.x >> 6, l = threadIdx.x & 63;
  MfmaLdsSplit &L = lds[wv];
  for (int q = blockIdx.x; q < nitems; q += gridDim.x) {
    const AxItem it = items[q];
    const BatchSolve &sd = sds[it.solve];
    DirMfma dir;
    if (batch_dir_mfma(sd, st, bd, it, dir)) continue;  // uniform per block
    m16x4 fh, fl, bh, bl;
    d_operands<N1>(l, (const uint16_t *)sd.D16hi, (const uint16_t *)sd.D16lo, fh,
                   fl, bh, bl);
    for (int e0 = 0; e0 < epb; e0 += MW) {  // uniform per block
      const int64_t e = it.elem0 + e0 + wv;
      // global pointers (their address space is not known from the descriptor)
      solve_elem_mfma<N1, SPLIT>(
          l, L, e, e0 + wv < epb && e < sd.E, bd.stream, sd.box, dir, (gp<float>)sd.v32[VWL],
          (const uint16_t *)sd.G16, (gp<const uint16_t>)sd.H16, fh, fl, bh, bl,
          (gp<double>)sd.edot);
      wave_lds_sync();  // L is reused by the next element
    }
  }
}

// The same operator for a single solve, every argument passed in (no work
// item or descriptor to fetch first), one element per wave; a finished
// solve's workgroups return at once.
template <int N1, bool SPLIT>
__global__ void __launch_bounds__(64 * MW)
    k_ax_mfma_solve(int64_t e0, int64_t E, const uint16_t *__restrict__ Dhi,
                    const uint16_t *__restrict__ Dlo, const uint16_t *__restrict__ G,
                    const uint16_t *__restrict__ H, const float *__restrict__ z,
                    float *__restrict__ w, Box box, DirArgs<float> da, int mode, int nt,
                    double *__restrict__ edot) {
  __shared__ MfmaLdsSplit lds[MW];
  const int wv = threadIdx.x >> 6, l = threadIdx.x & 63;
  DirMfma dir;
  dir.z = (gp<const float>)z;
  dir.p = (gp<const float>)da.p;
  dir.pnew = (gp<float>)da.pnew;
  if (dir_mfma(da.st, mode, da.part, da.stride, da.beg, da.end,
               e0 == 0 && blockIdx.x == 0 && threadIdx.x == 0, dir))
    return;  // uniform: the solve has ended
  m16x4 fh, fl, bh, bl;
  d_operands<N1>(l, Dhi, Dlo, fh, fl, bh, bl);
  const int64_t e = e0 + (int64_t)blockIdx.x * MW + wv;
  solve_elem_mfma<N1, SPLIT>(l, lds[wv], e, e < E, nt != 0, box, dir, (gp<float>)w, G,
                             (gp<const uint16_t>)H, fh, fl, bh, bl, (gp<double>)edot);
}

// one element of the solvers' operator at n1 = 9 (as solve_elem_mfma)
template <bool SPLIT>
__device__ inline void solve_elem_mfma9(int l, MfmaLds9 &L, int64_t e, bool act,
                                        const Box &box, const DirMfma &dir, gp<float> w,
                                        const uint16_t *G, gp<const uint16_t> H,
                                        m16x4 fh, m16x4 fl, m16x4 bh, m16x4 bl,
                                        gp<double> edot) {
  uint16_t gq[2][6][9];
  load_factors9(l, act, e, G, gq);
  constexpr int T9 = (E9 + 63) / 64;
  float pv[T9];  // p' at the lane's nodes p = l + 64 t
  gather_dir(
      box, dir, act, e,
      [&](int t, uint32_t &i, uint32_t &j, uint32_t &k) {
        const uint32_t p = l + 64 * t;
        i = p % 9, j = (p / 9) % 9, k = p / 81;
        return p < E9;
      },
      pv);
#pragma unroll
  for (int t = 0; t < T9; ++t) {
    const int p = l + 64 * t;
    if (p < E9) {
      const uint16_t hi = f32_to_bf16(pv[t]);
      L.u[p] = hi;
      L.ul[p] = f32_to_bf16(pv[t] - bf16_to_f32(hi));
    }
  }
  wave_lds_sync();
  mfma_element9<SPLIT, true>(l, L, gq, fh, fl, bh, bl);
  auto wval = [&](int p) {  // w at node p, as stored (mass term added)
    float v = L.gr[p];
    if (H != nullptr)
      v += bf16_to_f32(H[e * E9 + p]) * (bf16_to_f32(L.u[p]) + bf16_to_f32(L.ul[p]));
    return v;
  };
  if (act) {
    for (int p = l; p < E9; p += 64) w[e * E9 + p] = wval(p);
  }
  // each lane's nodes in ascending t, then the lanes (wval reads H at the
  // element)
  double cd = 0.0;
#pragma unroll
  for (int t = 0; t < T9; ++t)
    if (act && l + 64 * t < E9) cd += (double)pv[t] * (double)wval(l + 64 * t);
  cd = wave_sum(cd);
  if (act && l == 0) edot[e] = cd;
}

// the batched solver operator at n1 = 9: as k_bax_mfma, MW9 elements per
// workgroup pass
template <bool SPLIT>
__global__ void __launch_bounds__(64 * MW9) __attribute__((amdgpu_waves_per_eu(2)))
    k_bax_mfma9(const BatchSolve *__restrict__ sds, CgState *st,
                const AxItem *__restrict__ items, int nitems, int epb, BaxDir bd) {
  __shared__ MfmaLds9 lds[MW9];
  const int wv = threadIdx.x >> 6, l = threadIdx.x & 63;
  MfmaLds9 &L = lds[wv];
  for (int q = blockIdx.x; q < nitems; q += gridDim.x) {
    const AxItem it = items[q];
    const BatchSolve &sd = sds[it.solve];
    DirMfma dir;
    if (batch_dir_mfma(sd, st, bd, it, dir)) continue;  // uniform per block
    m16x4 fh, fl, bh, bl;
    d_operands9(l, (const uint16_t *)sd.D16hi, (const uint16_t *)sd.D16lo, fh, fl,
                bh, bl);
    for (int e0 = 0; e0 < epb; e0 += MW9) {  // uniform per block
      const int64_t e = it.elem0 + e0 + wv;
      // the lane number by a value the compiler cannot see through: it moved the
      // element routine's lane addresses and masks out of this loop, which took
      // 280 registers, one wave per SIMD (8 refinements of 9^3, N = 8, 96
      // iterations: 24.1 -> 16.7 ms)
      int le = l;
      asm volatile("" : "+v"(le));
      solve_elem_mfma9<SPLIT>(
          le, L, e, e0 + wv < epb && e < sd.E, sd.box, dir, (gp<float>)sd.v32[VWL],
          (const uint16_t *)sd.G16, (gp<const uint16_t>)sd.H16, fh, fl, bh, bl,
          (gp<double>)sd.edot);
      wave_lds_sync();  // L is reused by the next element
    }
  }
}

// the single-solve operator at n1 = 9 (as k_ax_mfma_solve)
template <bool SPLIT>
__global__ void __launch_bounds__(64 * MW9)
    k_ax_mfma_solve9(int64_t e0, int64_t E, const uint16_t *__restrict__ Dhi,
                     const uint16_t *__restrict__ Dlo, const uint16_t *__restrict__ G,
                     const uint16_t *__restrict__ H, const float *__restrict__ z,
                     float *__restrict__ w, Box box, DirArgs<float> da, int mode, int nt,
                     double *__restrict__ edot) {
  __shared__ MfmaLds9 lds[MW9];
  const int wv = threadIdx.x >> 6, l = threadIdx.x & 63;
  DirMfma dir;
  dir.z = (gp<const float>)z;
  dir.p = (gp<const float>)da.p;
  dir.pnew = (gp<float>)da.pnew;
  if (dir_mfma(da.st, mode, da.part, da.stride, da.beg, da.end,
               e0 == 0 && blockIdx.x == 0 && threadIdx.x == 0, dir))
    return;  // uniform: the solve has ended
  m16x4 fh, fl, bh, bl;
  d_operands9(l, Dhi, Dlo, fh, fl, bh, bl);
  const int64_t e = e0 + (int64_t)blockIdx.x * MW9 + wv;
  solve_elem_mfma9<SPLIT>(l, lds[wv], e, e < E, box, dir, (gp<float>)w, G,
                          (gp<const uint16_t>)H, fh, fl, bh, bl, (gp<double>)edot);
}

void launch_ax_mfma_solve(const SolveAx &a, hipStream_t s) {
  if (a.E <= 0) return;
  if (a.mode == 0) fail(SEM_ERR_ARG, "solve: the matrix-core operator runs inside CG only");
  const int n1 = a.N + 1;
  const bool split = a.prec == SEM_BF16_MFMA;
  const int nt = a.regime == AX_STREAM;
  const DirArgs<float> da = {(const float *)a.p, a.mode == 3 ? nullptr : (float *)a.pnew,
                             a.st,               a.part,
                             a.nparts,           0,
                             a.nparts};
  auto go = [&](auto kernel, int waves) {
    for (int64_t e0 = 0; e0 < a.E; e0 += MFMA_PIECE) {
      const int64_t n = std::min(a.E - e0, MFMA_PIECE);
      hipLaunchKernelGGL(kernel, dim3((unsigned)((n + waves - 1) / waves)), dim3(64 * waves), 0,
                         s, e0, a.E, (const uint16_t *)a.D, (const uint16_t *)a.Dlo,
                         (const uint16_t *)a.G, (const uint16_t *)a.H, (const float *)a.u,
                         (float *)a.w, a.box, da, a.mode, nt, a.edot);
    }
  };
  switch (n1) {
#define SEM_AXMS(NN)                          \
  case NN:                                    \
    if (split)                                \
      go(k_ax_mfma_solve<NN, true>, MW);      \
    else                                      \
      go(k_ax_mfma_solve<NN, false>, MW);     \
    break;
    SEM_AXMS(2)
    SEM_AXMS(3)
    SEM_AXMS(4)
    SEM_AXMS(5)
    SEM_AXMS(6)
    SEM_AXMS(7)
    SEM_AXMS(8)
#undef SEM_AXMS
    case 9:
      if (split)
        go(k_ax_mfma_solve9<true>, MW9);
      else
        go(k_ax_mfma_solve9<false>, MW9);
      break;
    default:
      fail(SEM_ERR_ARG, "solve: the matrix-core operator needs N in 1..8");
  }
  SEM_HIP(hipGetLastError());
}

void launch_bax_mfma(int n1, bool split, const BatchSolve *sds, CgState *st,
                     const AxItem *items, int nitems, int epb, int grid, const BaxDir &bd,
                     hipStream_t s) {
  if (nitems <= 0) return;
  if (bd.mode == 0) fail(SEM_ERR_ARG, "solve: the matrix-core operator runs inside CG only");
  auto go = [&](auto kernel, int waves) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(64 * waves), 0, s, sds, st, items,
                       nitems, epb, bd);
  };
  switch (n1) {
#define SEM_BAXM(NN)                     \
  case NN:                               \
    if (split)                           \
      go(k_bax_mfma<NN, true>, MW);      \
    else                                 \
      go(k_bax_mfma<NN, false>, MW);     \
    break;
    SEM_BAXM(2)
    SEM_BAXM(3)
    SEM_BAXM(4)
    SEM_BAXM(5)
    SEM_BAXM(6)
    SEM_BAXM(7)
    SEM_BAXM(8)
#undef SEM_BAXM
    case 9:
      if (split)
        go(k_bax_mfma9<true>, MW9);
      else
        go(k_bax_mfma9<false>, MW9);
      break;
    default:
      fail(SEM_ERR_ARG, "batched operator: the matrix-core operator needs N in 1..8");
  }
  SEM_HIP(hipGetLastError());
}

}  // namespace sem
