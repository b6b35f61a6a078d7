// The gathered operator of a single solve, w_L = A_L Q p_G (paper section
// 4.2.1 operator, applied inside the PCG of section 4.2.2): the element
// routine of the standalone operator with GATHER on, every pointer, the
// closed-form box numbering and the solver's done flag passed as kernel
// arguments.  A workgroup then issues its data loads at once; the batched
// kernel first has to fetch its work item and the solve's descriptor, a
// chain of dependent loads that cost ~25 % of the operator time at 32^3,
// N = 7 (measured with and without the gather: the gather itself costs
// nothing in FP64).  A mesh with a mass term passes H = alpha(X) B and the
// kernel adds H o u.  Inside an iteration (DIR 1 to 3) the kernel also stores
// every element's energy p_e^T w_e (the element terms of (p, A p), in an order
// fixed by the node indices); outside (DIR 0, the residuals) it runs in FP64.
// Workgroup shapes, load hints and the numbering of the element blocks over
// the XCDs: OpShape with SOLVE, which differ from the standalone operator's.
// NTW (a solve whose vectors exceed the last-level cache):
// the output is stored non-temporally: 188 -> 182 us FP64 at 32^3, N = 7, and
// the assembly that reads it next got faster too (FP32 56 -> 52 us).
#include "ax_tile.h"

namespace sem {

// threads: whole waves where the direction's scalars are formed by waves
template <int N1, class TG, int REG, int DIR> constexpr int solve_threads() {
  constexpr int T = OpShape<N1, sizeof(TG), true, REG>::THREADS;
  return DIR != 0 ? (T + 63) / 64 * 64 : T;
}

template <int N1, class TV, class TG, class TC, bool MASS, bool NTW, int REG, int DIR>
__global__ void __launch_bounds__((solve_threads<N1, TG, REG, DIR>()))
    k_ax_solve(int64_t E, const TC *__restrict__ D, const TG *__restrict__ G,
               const TV *__restrict__ u, TV *__restrict__ w, Box box,
               const TG *__restrict__ H, double *__restrict__ edot, DirArgs<TV> dir) {
  using S = OpShape<N1, sizeof(TG), true, REG>;
  __shared__ __align__(16) TC smem[lds_words<N1, TC>(S::EPB)];
  ax_tile<N1, S::EPB, TV, TG, TV, TC, true, NTW, MASS, S::NTG, DIR != 0, S::PRED, DIR>(
      threadIdx.x,
      // (the fused direction gathers twice and stores: runs per XCD at any size,
      // FP32 N = 3, 8M nodes 115 -> 109 us an iteration)
      (S::XCD || DIR == 1 ? xcd_run_block(blockIdx.x, gridDim.x) : (int64_t)blockIdx.x) *
          S::EPB,
      E, D, G, u, w, &box, smem, H, edot, DIR != 0 ? &dir : nullptr);
}

template <int N1, class TV, class TG, class TC, bool MASS, bool NTW, int REG, int DIR>
static void launch_solve_d(const SolveAx &a, hipStream_t s) {
  using S = OpShape<N1, sizeof(TG), true, REG>;
  const int64_t blocks = (a.E + S::EPB - 1) / S::EPB;
  if (blocks == 0) return;
  const DirArgs<TV> dir = {(const TV *)a.p, (TV *)a.pnew, a.st, a.part, a.nparts, 0, a.nparts};
  hipLaunchKernelGGL((k_ax_solve<N1, TV, TG, TC, MASS, NTW, REG, DIR>), dim3((unsigned)blocks),
                     dim3(solve_threads<N1, TG, REG, DIR>()), 0, s, a.E, (const TC *)a.D,
                     (const TG *)a.G, (const TV *)a.u, (TV *)a.w, a.box, (const TG *)a.H,
                     a.edot, dir);
}

template <int N1, class TV, class TG, class TC, bool MASS>
static void launch_solve_m(const SolveAx &a, hipStream_t s) {
  // the sums are added in the operator on few elements only, and a pass of its
  // own forms the direction where the vectors stream
  const bool stream = a.regime == AX_STREAM;
  if (a.mode == 2 && a.regime == AX_SMALL)
    launch_solve_d<N1, TV, TG, TC, MASS, false, AX_SMALL, 2>(a, s);
  else if (a.mode == 2)
    launch_solve_d<N1, TV, TG, TC, MASS, false, AX_CACHED, 2>(a, s);
  else if (a.mode == 1 && stream)
    launch_solve_d<N1, TV, TG, TC, MASS, false, AX_STREAM, 1>(a, s);
  else if (a.mode == 1)
    launch_solve_d<N1, TV, TG, TC, MASS, false, AX_CACHED, 1>(a, s);
  else if (a.mode == 3)
    launch_solve_d<N1, TV, TG, TC, MASS, true, AX_STREAM, 3>(a, s);
  else if constexpr (sizeof(TV) == 8) {  // the residuals: FP64
    if (stream)
      launch_solve_d<N1, TV, TG, TC, MASS, true, AX_STREAM, 0>(a, s);
    else
      launch_solve_d<N1, TV, TG, TC, MASS, false, AX_CACHED, 0>(a, s);
  } else {
    fail(SEM_ERR_ARG, "solve: the operator outside an iteration is FP64");
  }
}

template <int N1, class TV, class TG, class TC>
static void launch_solve_t(const SolveAx &a, hipStream_t s) {
  if (a.H != nullptr)
    launch_solve_m<N1, TV, TG, TC, true>(a, s);
  else
    launch_solve_m<N1, TV, TG, TC, false>(a, s);
}

template <int N1> static void launch_solve_n(const SolveAx &a, hipStream_t s) {
  if (a.prec == SEM_FP64)
    launch_solve_t<N1, double, double, double>(a, s);
  else if (a.prec == SEM_FP32)
    launch_solve_t<N1, float, float, float>(a, s);
  else
    launch_solve_t<N1, float, uint16_t, float>(a, s);
}

void launch_ax_solve(const SolveAx &a, hipStream_t s) {
  switch (a.N) {
    case 1: launch_solve_n<2>(a, s); break;
    case 2: launch_solve_n<3>(a, s); break;
    case 3: launch_solve_n<4>(a, s); break;
    case 4: launch_solve_n<5>(a, s); break;
    case 5: launch_solve_n<6>(a, s); break;
    case 6: launch_solve_n<7>(a, s); break;
    case 7: launch_solve_n<8>(a, s); break;
    case 8: launch_solve_n<9>(a, s); break;
    default: fail(SEM_ERR_ARG, "solve: N must be in 1..8");
  }
  SEM_HIP(hipGetLastError());
}

}  // namespace sem
