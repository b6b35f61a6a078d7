// The gathered operator of a single solve, w_L = A_L Q p_G (paper section
// 4.2.1 operator, applied inside the PCG of section 4.2.2): the element
// routine of the standalone operator with GATHER on, every pointer, the
// closed-form box numbering and the solver's done flag passed as kernel
// arguments.  A workgroup then issues its data loads at once; the batched
// kernel first has to fetch its work item and the solve's descriptor, a
// chain of dependent loads that cost ~25 % of the operator time at 32^3,
// N = 7 (measured with and without the gather: the gather itself costs
// nothing in FP64).  Workgroup shapes and load hints as the standalone
// operator (OpShape).  A mesh with
// a mass term passes H = alpha(X) B and the kernel adds H o u.  With edot
// non-null the kernel also stores every element's energy p_e^T w_e (the
// element terms of (p, A p), in an order fixed by the node indices).
// Workgroups are dealt to the 8 XCDs in turn (workgroup b runs on XCD
// b % 8), each with its own L2.  With FP32 / BF16 storage the kernel numbers
// its element blocks so that every XCD gets one contiguous run of them, and
// elements that share nodes of the gathered vector (neighbours along x, y
// and z) read the shared cache lines through the same L2: 102 -> 94 us at
// 32^3, N = 7, FP32.  In FP64 the same order was slower (181 -> 186 us), so
// FP64 keeps the plain order.  NTW (a solve whose vectors exceed the
// last-level cache): the output is stored non-temporally, as in the
// standalone operator: 188 -> 182 us FP64 at 32^3, N = 7, and the assembly
// that reads it next got faster too (FP32 56 -> 52 us).
#include "ax_tile.h"

namespace sem {

// element block of workgroup b of nb: XCD x = b % 8 takes the run
// [x q + min(x, r), ...) of q or q + 1 blocks (q = nb / 8, r = nb % 8)
__device__ inline int64_t xcd_run_block(unsigned b, unsigned nb) {
  const unsigned q = nb / 8, r = nb % 8, x = b % 8, k = b / 8;
  return (int64_t)x * q + (x < r ? x : r) + k;
}

// threads: whole waves where the direction's scalars are formed by waves
template <int N1, class TC, int DIR> constexpr int solve_threads() {
  constexpr int T = OpShape<N1, sizeof(TC)>::THREADS;
  return DIR != 0 ? (T + 63) / 64 * 64 : T;
}

template <int N1, class TV, class TG, class TC, bool MASS, bool NTW, int DIR>
__global__ void __launch_bounds__((solve_threads<N1, TC, DIR>()))
    k_ax_solve(int64_t E, const TC *__restrict__ D, const TG *__restrict__ G,
               const TV *__restrict__ u, TV *__restrict__ w, Box box,
               const TG *__restrict__ H, double *__restrict__ edot, DirArgs<TV> dir) {
  using S = OpShape<N1, sizeof(TC)>;
  __shared__ __align__(16) TC smem[lds_words<N1, TC>(S::EPB)];
  ax_tile<N1, S::EPB, TV, TG, TV, TC, true, NTW, MASS, S::NTG, DIR != 0, S::PRED, DIR>(
      threadIdx.x,
      (sizeof(TV) == 4 ? xcd_run_block(blockIdx.x, gridDim.x) : (int64_t)blockIdx.x) *
          S::EPB,
      E, D, G, u, w, &box, smem, H, edot, DIR != 0 ? &dir : nullptr);
}

template <int N1, class TV, class TG, class TC, bool MASS, bool NTW, int DIR>
static void launch_solve_d(const SolveAx &a, hipStream_t s) {
  using S = OpShape<N1, sizeof(TC)>;
  const int64_t blocks = (a.E + S::EPB - 1) / S::EPB;
  if (blocks == 0) return;
  const DirArgs<TV> dir = {(const TV *)a.p, (TV *)a.pnew, a.st, a.part, a.nparts, 0, a.nparts};
  hipLaunchKernelGGL((k_ax_solve<N1, TV, TG, TC, MASS, NTW, DIR>), dim3((unsigned)blocks),
                     dim3(solve_threads<N1, TC, DIR>()), 0, s, a.E, (const TC *)a.D,
                     (const TG *)a.G, (const TV *)a.u, (TV *)a.w, a.box, (const TG *)a.H,
                     a.edot, dir);
}

template <int N1, class TV, class TG, class TC, bool MASS>
static void launch_solve_m(const SolveAx &a, hipStream_t s) {
  // the direction is formed in the operator only where the vectors do not
  // stream, and in a pass of its own where they do
  if (a.mode == 2)
    launch_solve_d<N1, TV, TG, TC, MASS, false, 2>(a, s);
  else if (a.mode == 1)
    launch_solve_d<N1, TV, TG, TC, MASS, false, 1>(a, s);
  else if (a.mode == 3)
    launch_solve_d<N1, TV, TG, TC, MASS, true, 3>(a, s);
  else if (a.nt)
    launch_solve_d<N1, TV, TG, TC, MASS, true, 0>(a, s);
  else
    launch_solve_d<N1, TV, TG, TC, MASS, false, 0>(a, s);
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
