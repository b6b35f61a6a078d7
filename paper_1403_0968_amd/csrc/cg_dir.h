// The search direction inside the operator kernels of the CG iteration
// (paper section 4.2.2), for solves whose vectors stay in the caches.  An
// iteration is two passes over the data:
//   operator:  beta and the convergence test from the partial sums of the
//              last r update, p' = z + beta p at the gather, w_L = A_L Q p',
//              element energies of (p', A p');
//   r update:  alpha from the energies, x += alpha p', r -= alpha Q^T w_L,
//              z = dinv r, partial sums of (r, z) and (r, r).
// p' is stored once per unique node, by the first (lowest) element that
// holds the node, into a second buffer: other elements still read the old p
// of the nodes they share.  The form with a pass of its own for p and x and
// two scalar kernels is five launches; it moves the same bytes (the gather
// reads shared nodes of p and z again where the separate pass read and wrote
// them once) and is kept for vectors beyond the last-level cache, where the
// passes run at the memory's rate and the fused one is slower (FP64, 32^3,
// N = 7: operator 179 -> 212 us, r update 83 -> 136 us, against 66 us for
// the p and x pass).  In the caches the launches and their latency bound the
// iteration.  Solve times, five launches against two: FP64 4^3 N = 4 2.06 ->
// 1.34 ms, BF16 refinement 15 x 11 x 13 N = 7 37.1 -> 29.5 ms (27 -> 22 us per
// iteration); with the coarse correction at 24^3, N = 7, FP32 (where beta has
// its own kernel) 151 -> 148 ms.  (With the operator's size classes since: 1.27
// and 29.1 ms, and 133 ms with fewer terms in beta's kernel.)  Results are the
// same bits.
//
// Scalars are split so that no kernel writes what its other workgroups
// read: the operator reads the main fields of CgState and its first
// workgroup writes the *_b fields; the r update reads the *_b fields and its
// first workgroup writes the main ones.
//
// RED = true: every wave (operator) or workgroup (r update) adds up the
// partial sums itself, in the order the scalar kernels k_bbeta and
// k_balpha_e use, so both forms give the same bits; RED = false: the scalar
// kernels have run and the result is read from the state.
#pragma once

#include "common.h"
#include "sem_internal.h"

namespace sem {

// threads of the scalar kernels whose summation orders are reproduced here
constexpr int BT = 256;   // k_bbeta: (r, z), (r, r)
constexpr int AT = 1024;  // k_balpha_e: element energies

// what the operator needs to form p' of one solve
template <class TV> struct DirArgs {
  const TV *p;         // the last direction
  TV *pnew;            // the new one
  CgState *st;
  const double *part;  // rows of (r, z) and (r, r) partials, stride apart
  int32_t stride, beg, end;
};

// the outcome of one iteration's sums: state after the r update that
// produced them
__device__ inline int cg_verdict(double rz, double rr, double tol2, double bb, int it,
                                 int maxit) {
  if (!isfinite(rr) || !isfinite(rz)) return 2;
  if (rr <= tol2 * bb) return 1;
  if (it >= maxit) return 3;
  return 0;
}

// The scalars of one solve as the operator reads them: loaded before the
// element's data, so that their latency is hidden behind it.
struct DirScalars {
  double rz, rr, beta, tol2, bb;
  int done, it, ready, maxit;
};
__device__ inline DirScalars dir_scalars(const CgState *st_) {
  const gp<const CgState> st = (gp<const CgState>)st_;
  return {st->rz, st->rr, st->beta, st->tol2, st->bb, st->done, st->it, st->ready, st->maxit};
}

// The partial sums of a solve (at most RED_PARTS per row), loaded by one
// wave: lane l takes the entries of the threads l, l + 64, ... of k_bbeta's
// workgroup, all in flight at once.
constexpr int RED_PF = 4, RED_PARTS = RED_PF * BT;
template <bool RED> struct DirParts {
  static constexpr int V = RED ? BT / 64 : 1, P = RED ? RED_PF : 1;
  double a[P][V], b[P][V];
  __device__ void load(const double *part, int stride, int beg, int end) {
    if constexpr (RED) {
      const gp<const double> p = (gp<const double>)part;
      const int l = threadIdx.x & 63;
#pragma unroll
      for (int u = 0; u < P; ++u)
#pragma unroll
        for (int m = 0; m < V; ++m) {
          const int q = beg + u * BT + 64 * m + l;
          a[u][m] = q < end ? p[q] : 0.0;
          b[u][m] = q < end ? p[stride + q] : 0.0;
        }
    }
  }
  // each of k_bbeta's threads adds its entries in order, then the four
  // 64-thread sums are added as block_sum adds them
  __device__ void sums(double &rz, double &rr) const {
    rz = rr = 0.0;
#pragma unroll
    for (int m = 0; m < V; ++m) {
      double x = 0.0, y = 0.0;
#pragma unroll
      for (int u = 0; u < P; ++u) {
        x += a[u][m];
        y += b[u][m];
      }
      rz += wave_sum(x);
      rr += wave_sum(y);
    }
  }
};

struct DirStep {
  double beta;
  bool first;  // p' = z (no earlier direction)
  bool stop;   // the solve has ended
};

// the direction's step, the same in every lane; all 64 lanes of the wave
// must call it.  writer: this thread records the step for the r update.
template <bool RED>
__device__ inline DirStep dir_step(CgState *st, const DirScalars &s, const DirParts<RED> &parts,
                                   bool writer) {
  int done = s.done, it = s.it;
  double rz = s.rz, rr = s.rr, beta = s.beta;
  if constexpr (RED) {
    if (done == 0 && s.ready == 0) {  // uniform
      double nrz, nrr;
      parts.sums(nrz, nrr);
      it += 1;
      done = cg_verdict(nrz, nrr, s.tol2, s.bb, it, s.maxit);
      rr = nrr;
      if (done == 0) {
        beta = nrz / rz;
        rz = nrz;
      }
    }
  }
  if (writer) {
    const gp<CgState> w = (gp<CgState>)st;
    w->rz_b = rz;
    w->rr_b = rr;
    w->it_b = it;
    w->done_b = done;
  }
  return {beta, s.ready == 2, done != 0};
}

// a x + y rounded once.  The vector updates of the iteration are written with
// it: left to the compiler, the product z + beta p was contracted in one kernel
// and, moved into the branch that loads p, rounded by itself in another, and a
// solve's bits depended on the kernel (matrix-core refinement at N = 1, 2,
// alone against in a batch).
__device__ inline double axpy1(double a, double x, double y) { return __builtin_fma(a, x, y); }
__device__ inline float axpy1(float a, float x, float y) { return __builtin_fmaf(a, x, y); }

// whether an element at c stores the value of its node (i, j, k): the first
// element along each direction does (the coordinate that wraps to 0 belongs
// to element 0)
__device__ inline bool owns_coord(uint32_t node, uint32_t elem, uint32_t coord) {
  return node == 0 ? elem == 0 : coord != 0;
}

// The energies of a solve's elements (at most RED_ENERGIES), loaded by a
// workgroup of BT threads, all in flight at once, and their sum in
// k_balpha_e's order (AT threads, then their waves); every thread gets it.
constexpr int RED_EF = 4, RED_ENERGIES = RED_EF * AT;
template <bool RED> struct Energies {
  static constexpr int V = RED ? AT / BT : 1, P = RED ? RED_EF : 1;
  double v[P][V];
  __device__ void load(const double *edot, int64_t E) {
    if constexpr (RED) {
      const gp<const double> ed = (gp<const double>)edot;
#pragma unroll
      for (int u = 0; u < P; ++u)
#pragma unroll
        for (int m = 0; m < V; ++m) {
          const int q = u * AT + m * BT + (int)threadIdx.x;
          v[u][m] = q < E ? ed[q] : 0.0;
        }
    }
  }
  __device__ double sum(double *sm /* AT / 64 */) const {
    const int w = threadIdx.x >> 6;
#pragma unroll
    for (int m = 0; m < V; ++m) {
      double a = 0.0;
#pragma unroll
      for (int u = 0; u < P; ++u) a += v[u][m];
      a = wave_sum(a);
      if ((threadIdx.x & 63) == 0) sm[m * (BT / 64) + w] = a;
    }
    __syncthreads();
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < AT / 64; ++q) s += sm[q];
    return s;
  }
};

}  // namespace sem
