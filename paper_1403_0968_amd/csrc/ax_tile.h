// Element routine of the local stiffness action w = D^T G D u (paper
// section 4.2.1), shared by the operator kernels and the element-local
// solves of the learned correction.
//
// One thread per (i,j) column of an element holds the n1 values along k in
// registers (the t-direction contractions never leave registers); the r- and
// s-direction contractions read the current k-slice from LDS (row pitch
// n1+1, so the 8 distinct rows a wave reads at once sit in different banks).
// All loads of an element (its u column and the 6 n1 geometric factors of
// the column) are issued before any arithmetic.  Storage/compute types:
// FP64 (double everywhere), FP32, and BF16 (u and G bfloat16, D, arithmetic
// and w FP32; at n1 = 8 the BF16 factors are stored column-contiguous
// [E][6][n1^2][n1] and the BF16 input is read in 16-byte rows and
// redistributed through LDS).  GATHER = true reads u from a unique-node
// vector through the closed-form box numbering.  MASS = true adds the lumped
// mass term H o u (H = alpha(X) B, one value per local node in the storage
// type of G, natural [E][n1^3] layout: a wave's load of one k-slice is
// contiguous).
#pragma once

#include <type_traits>

#include "cg_dir.h"
#include "common.h"
#include "sem_internal.h"

namespace sem {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

template <class P> __device__ inline auto ld_stream(P p) {
  return __builtin_nontemporal_load(p);
}

// the value of lane `lane` of a wave
__device__ inline double readlane_f64(double v, int lane) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)b, lane);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// LDS row pitch of the slice stacks: n1 + 1 (the 8 distinct rows a wave
// reads at once sit in different banks), or 12 for FP32 arithmetic at n1 =
// 8, where the r-direction rows are read as two 16-byte vectors: 16-byte
// aligned rows whose 8 starts 48 bytes apart cover all 32 banks once
template <int N1, class TC> constexpr int ax_pad() {
  return (N1 == 8 && sizeof(TC) == 4) ? 12 : N1 + 1;
}

template <int N1, class TC = double> constexpr int lds_words(int epb) {
  return 3 * epb * N1 * N1 * ax_pad<N1, TC>();
}

// Workgroup shape and load hints of the operator kernels per order, storage
// type of the factors and size of the mesh, each timed over orders, shapes and
// sizes of 0.06M to 16M local nodes (standalone operator: SOLVE = false; the
// solvers' gathered one: true).  What decides:
//  * AX_SMALL, at most 0.2M local nodes: the fewest elements that fill a wave,
//    so that the mesh spreads over the compute units (FP64 N = 7, 0.1M nodes
//    6.6 -> 5.2 us against four elements per workgroup).
//  * AX_CACHED, the arrays that come round again fit the last-level cache (at
//    n1 = 8 in the standalone operator without a band in the middle,
//    launch_mass in ax.hip): 256 MiB of what one application of the standalone
//    operator moves, or of a solve's operator and vectors (24^3, N = 7, FP32
//    flexible CG at 314 MB: 137 ms a solve with the streaming forms, 152 ms with
//    these): no streaming hints, which would make the next application miss
//    (FP64 N = 7, 4M nodes 44.3 -> 40.7 us, 5.2M nodes 58.2 -> 63.4; FP32 N = 7,
//    8M nodes 40.6 -> 38.1; BF16 N = 1, 2M nodes 20.1 -> 6.4), and in the
//    solvers element blocks numbered so that every XCD takes one contiguous run
//    of them (XCD): neighbours share the gathered vector's lines in one L2 (FP64
//    N = 6, 2.4M nodes 51.2 -> 41.6 us, FP32 N = 7, 2.5M 29.5 -> 20.5).
//  * AX_STREAM: the factors are read with the streaming hint only where a
//    factor column of a wave's load covers whole cache lines (n1 = 8; n1 = 4
//    in FP64; in the standalone operator also the other orders of NTG below).
//    Elsewhere the hint makes the neighbouring pieces of a line miss again:
//    16M nodes, BF16 N = 1, 2, 3, 4, 5, 6, 8: 154, 131, 71, 86, 75, 63, 84 ->
//    37, 78, 36, 56, 46, 48, 57 us; FP32 N = 1, 2, 4: 214, 150, 104 -> 81,
//    105, 95; solver, 12M nodes, FP64 N = 4 150 -> 134, N = 5 137 -> 130, FP32
//    N = 3 72 -> 57, N = 8 105 -> 76.  Contiguous runs per XCD are slower here
//    except for FP32 and BF16 at n1 = 8 (FP64 N = 5 130 -> 143, FP32 N = 5 72
//    -> 77; FP32 N = 7 74 -> 62).
// FP64 takes EPB elements per workgroup so that EPB n1^2 fills whole waves
// except where one wave per element was faster.  PRED: the loads carry the
// thread's element predicate instead of reading a valid stand-in element
// (FP64 at n1 = 7 and 9, where the unpredicated loads were 5-7 % slower;
// elsewhere they are faster, by 12 % at n1 = 2 and 16 % at n1 = 3).
constexpr int64_t AX_SMALL_NODES = 200000;
constexpr double AX_CACHE_BYTES = 256.0 * 1024 * 1024;
constexpr double SOLVE_CACHE_BYTES = 256.0 * 1024 * 1024;

// standalone operator; node_bytes: what one application moves per local node
inline AxRegime ax_regime(int64_t nodes, int node_bytes) {
  if (nodes <= AX_SMALL_NODES) return AX_SMALL;
  return (double)nodes * node_bytes <= AX_CACHE_BYTES ? AX_CACHED : AX_STREAM;
}
// solves of nL local and nG unique nodes in all: factors of gb and vectors of
// vb bytes a value, six vectors and the E-vector
inline double solve_bytes(int64_t nL, int64_t nG, int gb, int vb) {
  return (double)nL * (6 * gb + vb) + 6.0 * vb * (double)nG;
}
inline AxRegime solve_regime(int64_t nL, int64_t nG, int gb, int vb) {
  if (nL <= AX_SMALL_NODES) return AX_SMALL;
  return solve_bytes(nL, nG, gb, vb) <= SOLVE_CACHE_BYTES ? AX_CACHED : AX_STREAM;
}

template <int N1, int GB, bool SOLVE, int REG> struct OpShape {
  static constexpr int NP = N1 * N1;
  static constexpr int FILL = (64 / NP) > 0 ? 64 / NP : 1;
  static constexpr int pick(int a2, int a3, int a4, int a5, int a6, int a7, int a8, int a9) {
    return N1 == 2 ? a2 : N1 == 3 ? a3 : N1 == 4 ? a4 : N1 == 5 ? a5 : N1 == 6 ? a6
           : N1 == 7 ? a7 : N1 == 8 ? a8 : a9;
  }
  static constexpr int epb() {
    if (REG == AX_SMALL) return FILL;
    if (GB == 8 && !SOLVE) return pick(64, 7, 4, 5, 7, 5, 4, 3);
    if (GB == 8) return REG == AX_CACHED ? pick(64, 7, 4, 5, 7, 1, 1, 3)
                                         : pick(64, 7, 4, 5, 7, 1, 4, 3);
    if (SOLVE) return REG == AX_STREAM && GB == 4 ? pick(16, 14, 16, 5, 7, 1, 1, 3)
                                                  : pick(16, 14, 16, 5, 7, 5, 1, 3);
    if (GB == 4) return REG == AX_CACHED ? pick(16, 14, 4, 2, 3, 1, 1, 1)
                                         : pick(64, 28, 4, 2, 1, 1, 1, 1);
    return REG == AX_CACHED ? pick(16, 14, 4, 2, 3, 1, 1, 3) : pick(16, 14, 4, 5, 3, 5, 1, 3);
  }
  static constexpr bool ntg() {
    if (REG != AX_STREAM) return false;
    if (N1 == 8) return true;
    if (GB == 8 && SOLVE) return N1 == 4 || N1 == 7 || N1 == 9;
    if (GB == 8) return N1 == 4 || N1 == 6 || N1 == 7 || N1 == 9;
    return GB == 4 && !SOLVE && (N1 == 4 || N1 == 6 || N1 == 7);
  }
  static constexpr int EPB = epb();
  static constexpr int THREADS = EPB * NP;
  static constexpr bool NTG = ntg();
  static constexpr bool PRED = GB == 8 && (N1 == 9 || (N1 == 7 && EPB > 1));
  static constexpr bool XCD = SOLVE && (REG != AX_STREAM || (N1 == 8 && GB != 8));
};

// element block of workgroup b of nb: workgroups are dealt to the 8 XCDs in
// turn (workgroup b runs on XCD b % 8), each with its own L2; XCD x = b % 8
// takes the run [x q + min(x, r), ...) of q or q + 1 blocks (q = nb / 8, r =
// nb % 8)
__device__ inline int64_t xcd_run_block(unsigned b, unsigned nb) {
  const unsigned q = nb / 8, r = nb % 8, x = b % 8, k = b / 8;
  return (int64_t)x * q + (x < r ? x : r) + k;
}

// Apply the operator to elements e0 .. e0 + EPB - 1 (those < E) with the
// threads t = 0 .. of one workgroup; threads t >= EPB n1^2 only join the
// barriers.  smem holds 3 EPB n1^2 (n1+1) values of TC (8-byte aligned).
// EDOT = true also stores the element energy edot[e] = u_e^T w_e in FP64,
// summed in an order fixed by the node indices alone (each (i, j) column
// over k, then, at n1 = 8, the 64 column sums in registers by a fixed
// pattern over the lanes c = i + 8 j, otherwise the columns of a row j over
// i and then the rows over j), so that every tile shape gives the same bits.  Inside the solvers u is the
// search direction p, which vanishes on Dirichlet nodes, and the sum of the
// element energies is (p, A p) of the assembled operator.
// DIR != 0 (one CG iteration): nothing is stored once the solve has ended.
// DIR 3: u is the search direction.  DIR 1 or 2 (cg_dir.h): u is z, and the
// operator acts on p' = z + beta p, formed here and stored once per unique
// node; beta comes from the solve's state (1) or from the partial sums (2).
// All 64 lanes of every wave must then be launched.
template <int N1, int EPB, class TU, class TG, class TW, class TC, bool GATHER,
          bool NTW, bool MASS = false, bool NTG = true, bool EDOT = false,
          bool PRED = false, int DIR = 0, bool DESC = false>
__device__ __forceinline__ void ax_tile(int t, int64_t e0, int64_t E,
                                        const TC *__restrict__ D_,
                                        const TG *__restrict__ G_,
                                        const TU *__restrict__ u_,
                                        TW *__restrict__ w_,
                                        const Box *__restrict__ box,
                                        TC *__restrict__ smem,
                                        const TG *__restrict__ H_ = nullptr,
                                        double *__restrict__ edot_ = nullptr,
                                        const DirArgs<TU> *dir = nullptr) {
  static_assert(DIR == 0 || (GATHER && EDOT && sizeof(TU) == sizeof(TC)),
                "the direction is formed at the solvers' gather");
  // every array is global memory (the batched kernel reads these pointers
  // from a descriptor, where their address space is not known)
  // (DESC: D comes from a descriptor; 80 vector loads an element fewer, 64 ->
  // 47 us for 9 FP32 solves of 12^3, N = 7.  Single FP64 solves were 1 %
  // slower with it)
  typedef typename std::conditional<DESC, cp<TC>, gp<const TC>>::type DPtr;
  const DPtr D = (DPtr)D_;
  const gp<const TG> G = (gp<const TG>)G_;
  const gp<const TU> u = (gp<const TU>)u_;
  const gp<TW> w = (gp<TW>)w_;
  const gp<const TG> H = (gp<const TG>)H_;
  const gp<double> edot = (gp<double>)edot_;
  constexpr int NP = N1 * N1, N3 = N1 * NP, PAD = ax_pad<N1, TC>();
  // FP32 arithmetic at n1 = 8: the rows (k, j, 0..7) of s_u and s_r are
  // read as two 16-byte vectors
  constexpr bool VROW = PAD == 12;
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  constexpr int SL = N1 * N1 * PAD;  // one element's slice stack
  // n1 = 8: one element per wave (t is the thread index in the workgroup),
  // so the element index and the gather's box arithmetic are wave-uniform
  const int el = NP == 64 ? __builtin_amdgcn_readfirstlane(t / NP) : t / NP;
  const bool lane_ok = el < EPB;
  const int elc = lane_ok ? el : 0;
  const int c = t - el * NP;
  const int i = c % N1, j = c / N1;
  const int64_t e = e0 + el;
  const bool act = lane_ok && e < E;
  const int64_t base = e * N3 + c;
  // loads read element ed: e itself, or the workgroup's first element
  // (always < E) for threads without an element, so that no load needs a
  // predicate; only the stores are guarded.  PRED = true keeps a predicate
  // on every load instead (lanes without an element read nothing)
  const int64_t ed = act ? e : e0;
  const bool ld_on = !PRED || act;
  const int64_t based = ed * N3 + c;
  TC *s_u = smem + (0 * EPB + elc) * SL;
  TC *s_r = smem + (1 * EPB + elc) * SL;
  TC *s_s = smem + (2 * EPB + elc) * SL;
#define AX_IDX(k, jj, ii) (((k) * N1 + (jj)) * PAD + (ii))
  // n1 = 8: an element is one whole wave with its own slice stack, so the
  // phases of the element need only a wave-level barrier
  auto phase_sync = [] {
    if constexpr (NP == 64)
      wave_lds_sync();
    else
      __syncthreads();
  };

  constexpr bool VEC16 = sizeof(TG) == 2 && N1 == 8;  // BF16 column layout
  constexpr bool VECU = sizeof(TU) == 2 && N1 == 8 && !GATHER;
  constexpr bool FUSE = DIR == 1 || DIR == 2;
  // the solve's scalars and partial sums are asked for first and waited for
  // last: waiting for them before the element's loads are issued put a memory
  // round trip in front of every workgroup
  DirScalars dsc = {};
  DirParts<DIR == 2> dparts;
  if constexpr (DIR != 0) {
    if (dir != nullptr) {
      dsc = dir_scalars(dir->st);
      dparts.load(dir->part, dir->stride, dir->beg, dir->end);
    }
  }
  TU ucol[N1];
  TU pcol[FUSE ? N1 : 1];  // the old direction
  int64_t dg0 = 0, dgl = 0, dgs = 0;  // FUSE: the column's nodes are dg0 + dgs k, the last dgl
  bool own_c = false, own_0 = false, own_l = false;  // FUSE: nodes stored by this element
  u32x4 urow = {0u, 0u, 0u, 0u};
  if constexpr (VECU) {
    // lane c reads the 16-byte row (k, j) = (c / 8, c % 8) of the element
    urow = *(gp<const u32x4>)(u + ed * N3 + 8 * c);
  } else if constexpr (GATHER) {
    // the column's global (x, y) offset and the element's first z
    // coordinate; a coordinate E_d N of a periodic direction wraps to 0
    const ElemXYZ c3 = box_elem(*box, (uint32_t)ed);
    const uint32_t gx = wrap_coord(c3.x * (uint32_t)(N1 - 1) + i, box->Gx);
    const uint32_t gy = wrap_coord(c3.y * (uint32_t)(N1 - 1) + j, box->Gy);
    const int64_t gxy = (int64_t)gx + (int64_t)box->Gx * gy;
    const uint32_t gz0 = c3.z * (uint32_t)(N1 - 1);
    const int64_t Gxy = box->Gxy;
    // gz0 + k < G_z below the element's last z node: only that one wraps
    const int64_t g0 = gxy + Gxy * gz0;
#pragma unroll
    for (int k = 0; k < N1 - 1; ++k) ucol[k] = ld_on ? u[g0 + Gxy * k] : TU(0);
    const uint32_t gzl = wrap_coord(gz0 + N1 - 1, box->Gz);
    ucol[N1 - 1] = ld_on ? u[gxy + Gxy * gzl] : TU(0);
    if constexpr (FUSE) {
      const gp<const TU> po = (gp<const TU>)dir->p;
      dg0 = g0;
      dgl = gxy + Gxy * gzl;
      dgs = Gxy;
#pragma unroll
      for (int k = 0; k < N1 - 1; ++k) pcol[k] = ld_on ? po[g0 + Gxy * k] : TU(0);
      pcol[N1 - 1] = ld_on ? po[dgl] : TU(0);
      own_c = act && owns_coord(i, c3.x, gx) && owns_coord(j, c3.y, gy);
      own_0 = c3.z == 0;
      own_l = gzl != 0;
    }
  } else {
#pragma unroll
    for (int k = 0; k < N1; ++k) ucol[k] = ld_on ? u[based + k * NP] : TU(0);
  }
  TG g[6][N1];
  if constexpr (VEC16) {
#pragma unroll
    for (int q = 0; q < 6; ++q) {
      const gp<const u32x4> row = (gp<const u32x4>)(G + ed * 6 * N3 + q * N3 + 8 * c);
      const u32x4 v = NTG ? __builtin_nontemporal_load(row) : *row;
      const uint32_t wv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int h = 0; h < 4; ++h) {
        g[q][2 * h] = (TG)(wv[h] & 0xffffu);
        g[q][2 * h + 1] = (TG)(wv[h] >> 16);
      }
    }
  } else {
    const gp<const TG> Ge = G + ed * 6 * N3 + c;
#pragma unroll
    for (int k = 0; k < N1; ++k)
#pragma unroll
      for (int q = 0; q < 6; ++q)
        g[q][k] = !ld_on ? TG(0)
                  : NTG  ? ld_stream(Ge + q * N3 + k * NP)
                         : Ge[q * N3 + k * NP];
  }

  // (the mass factor is read with the streaming hint in every size class: the
  // rule of the factors, NTG, is not applied to it)
  TG hm[MASS ? N1 : 1];
  if constexpr (MASS) {
#pragma unroll
    for (int k = 0; k < N1; ++k) hm[k] = ld_on ? ld_stream(H + based + k * NP) : TG(0);
  }
  // every load above is issued before anything below: without the fence
  // the scheduler may wait for u (to store it into LDS) before it issues the
  // factor loads, which halves the bytes in flight (165 -> 201 us, FP64,
  // 32^3, N = 7)
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (DIR == 3) {
    // (no dir: the caller has looked)
    if (dir != nullptr && dsc.done != 0) return;  // uniform
  }
  if constexpr (FUSE) {
    const DirStep ds = dir_step<DIR == 2>(dir->st, dsc, dparts, t == 0 && e0 == 0);
    if (ds.stop) return;  // uniform
    const TU beta = (TU)ds.beta;
#pragma unroll
    for (int k = 0; k < N1; ++k) {
      // the first iteration has no old direction (its buffer may hold anything)
      if (!ds.first) ucol[k] = axpy1(beta, pcol[k], ucol[k]);
    }
    if (own_c) {
      const gp<TU> pn = (gp<TU>)dir->pnew;
#pragma unroll
      for (int k = 0; k < N1; ++k) {
        if (k == 0 ? own_0 : k == N1 - 1 ? own_l : true)
          pn[k == N1 - 1 ? dgl : dg0 + dgs * k] = ucol[k];
      }
    }
  }

  TC uc[N1];
  if constexpr (VECU) {
    const uint32_t wv[4] = {urow.x, urow.y, urow.z, urow.w};
    if (lane_ok) {
#pragma unroll
      for (int h = 0; h < 4; ++h) {
        s_u[AX_IDX(c / 8, c % 8, 2 * h)] = Cvt<TU, TC>::ld((TU)(wv[h] & 0xffffu));
        s_u[AX_IDX(c / 8, c % 8, 2 * h + 1)] = Cvt<TU, TC>::ld((TU)(wv[h] >> 16));
      }
    }
    phase_sync();
#pragma unroll
    for (int k = 0; k < N1; ++k) uc[k] = s_u[AX_IDX(k, j, i)];
  } else {
#pragma unroll
    for (int k = 0; k < N1; ++k) {
      uc[k] = Cvt<TU, TC>::ld(ucol[k]);
      if (lane_ok) s_u[AX_IDX(k, j, i)] = uc[k];
    }
  }
  // mass term H o u, formed while u is in registers; it starts the output sum
  TC mv[N1];
#pragma unroll
  for (int k = 0; k < N1; ++k) {
    if constexpr (MASS)
      mv[k] = Cvt<TG, TC>::ld(hm[k]) * uc[k];
    else
      mv[k] = TC(0);
  }
  TC Di[N1], Dj[N1];
#pragma unroll
  for (int m = 0; m < N1; ++m) {
    Di[m] = D[i * N1 + m];
    Dj[m] = D[j * N1 + m];
  }
  phase_sync();

  // gradient (r, s from LDS; t from registers) and fluxes, slice by slice
  TC wt[N1];
#pragma unroll
  for (int k = 0; k < N1; ++k) {
    TC ur = TC(0), us = TC(0), ut = TC(0);
    TC rowu[VROW ? N1 : 1];
    if constexpr (VROW) {
      const f32x4 a0 = *reinterpret_cast<const f32x4 *>(&s_u[AX_IDX(k, j, 0)]);
      const f32x4 a1 = *reinterpret_cast<const f32x4 *>(&s_u[AX_IDX(k, j, 4)]);
      rowu[0] = a0.x, rowu[1] = a0.y, rowu[2] = a0.z, rowu[3] = a0.w;
      rowu[4] = a1.x, rowu[5] = a1.y, rowu[6] = a1.z, rowu[7] = a1.w;
    }
#pragma unroll
    for (int m = 0; m < N1; ++m) {
      ur += Di[m] * (VROW ? rowu[VROW ? m : 0] : s_u[AX_IDX(k, j, m)]);
      us += Dj[m] * s_u[AX_IDX(k, m, i)];
      ut += D[k * N1 + m] * uc[m];
    }
    const TC g0 = Cvt<TG, TC>::ld(g[0][k]), g1 = Cvt<TG, TC>::ld(g[1][k]),
             g2 = Cvt<TG, TC>::ld(g[2][k]), g3 = Cvt<TG, TC>::ld(g[3][k]),
             g4 = Cvt<TG, TC>::ld(g[4][k]), g5 = Cvt<TG, TC>::ld(g[5][k]);
    if (lane_ok) {
      s_r[AX_IDX(k, j, i)] = g0 * ur + g1 * us + g2 * ut;
      s_s[AX_IDX(k, j, i)] = g1 * ur + g3 * us + g4 * ut;
    }
    wt[k] = g2 * ur + g4 * us + g5 * ut;
  }
  phase_sync();

  // w = D_r^T w_r + D_s^T w_s + D_t^T w_t
  TC DTi[N1], DTj[N1];
#pragma unroll
  for (int m = 0; m < N1; ++m) {
    DTi[m] = D[m * N1 + i];
    DTj[m] = D[m * N1 + j];
  }
  double cdot = 0.0;  // EDOT: this column's u^T w
#pragma unroll
  for (int k = 0; k < N1; ++k) {
    TC acc = mv[k];
    TC rowr[VROW ? N1 : 1];
    if constexpr (VROW) {
      const f32x4 a0 = *reinterpret_cast<const f32x4 *>(&s_r[AX_IDX(k, j, 0)]);
      const f32x4 a1 = *reinterpret_cast<const f32x4 *>(&s_r[AX_IDX(k, j, 4)]);
      rowr[0] = a0.x, rowr[1] = a0.y, rowr[2] = a0.z, rowr[3] = a0.w;
      rowr[4] = a1.x, rowr[5] = a1.y, rowr[6] = a1.z, rowr[7] = a1.w;
    }
#pragma unroll
    for (int m = 0; m < N1; ++m) {
      acc += DTi[m] * (VROW ? rowr[VROW ? m : 0] : s_r[AX_IDX(k, j, m)]);
      acc += DTj[m] * s_s[AX_IDX(k, m, i)];
      acc += D[m * N1 + k] * wt[m];
    }
    if constexpr (EDOT) cdot += (double)uc[k] * (double)(TW)acc;
    if (act) {
      if constexpr (NTW)
        __builtin_nontemporal_store((TW)acc, w + base + k * NP);
      else
        w[base + k * NP] = (TW)acc;
    }
  }
  if constexpr (EDOT && NP == 64) {
    // n1 = 8: every element is one whole wave (its 64 columns are the lanes
    // of a wave in every tile shape), so the column sums are added in
    // registers: lane exchanges within quads, then mirrored halves of each
    // 8 and 16 lanes (each step adds two equal-sized partial sums, and
    // a + b = b + a, so all lanes of a row hold the same bits), then the
    // four row sums in order
    double v = cdot;
    v += dpp_f64<0xB1>(v);   // quad_perm [1, 0, 3, 2]
    v += dpp_f64<0x4E>(v);   // quad_perm [2, 3, 0, 1]
    v += dpp_f64<0x141>(v);  // row_half_mirror
    v += dpp_f64<0x140>(v);  // row_mirror
    const double sum =
        ((readlane_f64(v, 0) + readlane_f64(v, 16)) + readlane_f64(v, 32)) + readlane_f64(v, 48);
    if (act && c == 0) edot[e] = sum;
  } else if constexpr (EDOT) {
    // s_u is no longer read after the barrier above: it holds the column
    // sums red[c] (c = i + n1 j) and then the row sums red[NP + j]
    double *red = reinterpret_cast<double *>(s_u);
    if (lane_ok) red[c] = cdot;
    __syncthreads();
    if (lane_ok && i == 0) {
      double r = 0.0;
#pragma unroll
      for (int ii = 0; ii < N1; ++ii) r += red[ii + N1 * j];
      red[NP + j] = r;
    }
    __syncthreads();
    if (act && c == 0) {
      double r = 0.0;
#pragma unroll
      for (int jj = 0; jj < N1; ++jj) r += red[NP + jj];
      edot[e] = r;
    }
  }
#undef AX_IDX
}

}  // namespace sem
