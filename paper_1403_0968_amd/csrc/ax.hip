// Local stiffness action w = D^T G D u on hexahedral spectral elements
// (paper section 4.2.1, factored stiffness operator with the G^T G metric
// precomputed per elemental node; section 4.2.2 names it the dominant cost of
// every PCG iteration).
//
// Kernel design for gfx950 (HBM-bound: 64 B per node in FP64 against ~111
// flops per node at N=7):
//   * one thread per (i,j) column of an element, holding the n1 values along
//     k in registers: the t-direction contractions never leave registers;
//   * the r- and s-direction contractions read the current k-slice from LDS
//     (row pitch n1+1 so that the 8 distinct rows a wave reads at once sit in
//     different banks);
//   * all loads of an element (its u column and the 6 n1 geometric factors of
//     the column) are issued before any arithmetic, so each wave keeps its
//     whole input in flight; factors and outputs of operators beyond the
//     last-level cache bypass the caches where whole lines are loaded
//     (OpShape);
//   * u, the r-flux and the s-flux each have their own LDS array.
// Storage/compute type combinations:
//   FP64: u, G, w double; FP32: float everywhere;
//   BF16: u and G bfloat16, D, arithmetic and w in FP32.  At n1 = 8 the BF16
//   factors are stored column-contiguous ([E][6][n1^2][n1]) so that a lane
//   fetches the 8 values of one factor with a single 16-byte load, and the
//   BF16 input is read in 16-byte rows and redistributed through LDS.
// GATHER = true reads u from a unique-node vector (the Q of the assembled
// operator), used inside the solvers; the unique index of each node comes
// from the closed-form box numbering, so the gather adds no index traffic
// and its loads issue with the others.  With a mass term (alpha != 0) the
// standalone operator also streams H = alpha(X) B and adds H o u (the lumped
// mass operator of equation semOperator): 72 B per node in FP64.
//
// Two kernels share one element routine: k_ax (one tile of elements per
// workgroup, the standalone operator) and k_bax (persistent workgroups
// walking a list of (solve, element tile) items of a batch of independent
// solves with mixed orders; one launch applies the operators of all solves,
// inside CG to the new direction p' = z + beta p formed at the gather
// (cg_dir.h), and stores every element's energy p'_e^T w_e for (p', A p')).
#include "ax_tile.h"

namespace sem {

// ---------------------------------------------------------------------------
// standalone operator: one tile per workgroup
// ---------------------------------------------------------------------------
template <int N1, class TU, class TG, class TW, class TC, bool MASS, int REG>
__global__ void __launch_bounds__((OpShape<N1, sizeof(TG), false, REG>::THREADS))
    k_ax(int64_t E, const TC *__restrict__ D, const TG *__restrict__ G,
         const TU *__restrict__ u, TW *__restrict__ w, const TG *__restrict__ H) {
  using S = OpShape<N1, sizeof(TG), false, REG>;
  __shared__ __align__(16) TC smem[lds_words<N1, TC>(S::EPB)];
  ax_tile<N1, S::EPB, TU, TG, TW, TC, false, REG == AX_STREAM, MASS, S::NTG, false, S::PRED>(
      threadIdx.x, (int64_t)blockIdx.x * S::EPB, E, D, G, u, w, nullptr, smem, H);
}

template <int N1, class TU, class TG, class TW, class TC, bool MASS, int REG>
static void launch_reg(int64_t E, const void *D, const void *G, const void *H,
                       const void *u, void *w, hipStream_t s) {
  using S = OpShape<N1, sizeof(TG), false, REG>;
  const int64_t blocks = (E + S::EPB - 1) / S::EPB;
  if (blocks == 0) return;
  hipLaunchKernelGGL((k_ax<N1, TU, TG, TW, TC, MASS, REG>), dim3((unsigned)blocks),
                     dim3(S::THREADS), 0, s, E, (const TC *)D, (const TG *)G,
                     (const TU *)u, (TW *)w, (const TG *)H);
}

template <int N1, class TU, class TG, class TW, class TC, bool MASS>
static void launch_mass(int64_t E, const void *D, const void *G, const void *H,
                        const void *u, void *w, hipStream_t s) {
  const int64_t nodes = E * N1 * N1 * N1;
  const int node_bytes = (int)((MASS ? 7 : 6) * sizeof(TG) + sizeof(TU) + sizeof(TW));
  AxRegime reg = ax_regime(nodes, node_bytes);
  // At n1 = 8, where the hint costs no partial lines, the streaming forms are
  // faster between the L2s' and half the last-level cache's size (FP64 58 MB
  // 12.7 -> 11.9 us, 83 MB 18.1 -> 17.8; FP32 64 MB 12.9 -> 11.3, 90 MB 16.6 ->
  // 15.7, 128 MB 21.4 -> 20.8; BF16 72 MB 17.4 -> 15.5), and slower on both
  // sides (FP64 38 MB 10.5 -> 11.4, 179 MB 32.6 -> 34.3; BF16 36 MB 9.0 -> 9.3,
  // 144 MB 26.8 -> 27.6)
  const double mib = (double)nodes * node_bytes / (1024.0 * 1024.0);
  if (N1 == 8 && reg == AX_CACHED && mib > 38.0 && mib <= 130.0) reg = AX_STREAM;
  if (reg == AX_SMALL)
    launch_reg<N1, TU, TG, TW, TC, MASS, AX_SMALL>(E, D, G, H, u, w, s);
  else if (reg == AX_CACHED)
    launch_reg<N1, TU, TG, TW, TC, MASS, AX_CACHED>(E, D, G, H, u, w, s);
  else
    launch_reg<N1, TU, TG, TW, TC, MASS, AX_STREAM>(E, D, G, H, u, w, s);
}

template <int N1, class TU, class TG, class TW, class TC>
static void launch_nt(int64_t E, const void *D, const void *G, const void *H,
                      const void *u, void *w, hipStream_t s) {
  if (H != nullptr)
    launch_mass<N1, TU, TG, TW, TC, true>(E, D, G, H, u, w, s);
  else
    launch_mass<N1, TU, TG, TW, TC, false>(E, D, G, H, u, w, s);
}

template <int N1>
static void launch_n(int prec, int64_t E, const void *D, const void *G,
                     const void *H, const void *u, void *w, hipStream_t s) {
  if (prec == SEM_FP64)
    launch_nt<N1, double, double, double, double>(E, D, G, H, u, w, s);
  else if (prec == SEM_FP32)
    launch_nt<N1, float, float, float, float>(E, D, G, H, u, w, s);
  else
    launch_nt<N1, uint16_t, uint16_t, float, float>(E, D, G, H, u, w, s);
}

void launch_ax(int N, int prec, int64_t E, const void *D, const void *G,
               const void *H, const void *u, void *w, hipStream_t s) {
  switch (N) {
    case 1: launch_n<2>(prec, E, D, G, H, u, w, s); break;
    case 2: launch_n<3>(prec, E, D, G, H, u, w, s); break;
    case 3: launch_n<4>(prec, E, D, G, H, u, w, s); break;
    case 4: launch_n<5>(prec, E, D, G, H, u, w, s); break;
    case 5: launch_n<6>(prec, E, D, G, H, u, w, s); break;
    case 6: launch_n<7>(prec, E, D, G, H, u, w, s); break;
    case 7: launch_n<8>(prec, E, D, G, H, u, w, s); break;
    case 8: launch_n<9>(prec, E, D, G, H, u, w, s); break;
    default: fail(SEM_ERR_ARG, "sem_ax: N must be in 1..8");
  }
  SEM_HIP(hipGetLastError());
}

// ---------------------------------------------------------------------------
// persistent batched operator: work items are (solve, first element) tiles;
// each workgroup walks items blockIdx.x, blockIdx.x + gridDim.x, ...
// ---------------------------------------------------------------------------
// elements per tile; launches with BS < N1^2 are refused (bax_min_block)
template <int BS, int N1> struct BTile {
  static constexpr int EPB = (BS / (N1 * N1)) > 0 ? BS / (N1 * N1) : 1;
};

// the direction arguments of a solve of the batch: the old direction in, the
// new one out; par selects which of VP and VW is which
template <class TV>
__device__ inline DirArgs<TV> batch_dir(const BatchSolve &sd, CgState *st, const BaxDir &bd,
                                        int s) {
  auto v = [&](int i) { return (TV *)(sizeof(TV) == 8 ? sd.v64[i] : sd.v32[i]); };
  return {v(bd.par ? VW : VP), v(bd.par ? VP : VW), st + s, bd.part, bd.stride,
          bd.vbeg[s],          bd.vbeg[s + 1]};
}

template <int BS, class TV, class TG, class TC, int DIR, bool STREAM, int N1>
__device__ __forceinline__ void bax_one(const BatchSolve &sd, int64_t e0, int src,
                                        const DirArgs<TV> &dir, TC *smem) {
  const TV *u = (const TV *)(sizeof(TV) == 8 ? sd.v64[src] : sd.v32[src]);
  TV *w = (TV *)(sizeof(TV) == 8 ? sd.v64[VWL] : sd.v32[VWL]);
  const TG *G = (const TG *)(sizeof(TG) == 8   ? sd.G64
                             : sizeof(TG) == 4 ? sd.G32
                                               : sd.G16);
  const TC *D = (const TC *)(sizeof(TC) == 8 ? sd.D64 : sd.D32);
  // hints as the single-solve operator's; with the vectors beyond the cache
  // the output streams non-temporally
  constexpr bool NTG = OpShape<N1, sizeof(TG), true, STREAM ? AX_STREAM : AX_CACHED>::NTG;
  ax_tile<N1, BTile<BS, N1>::EPB, TV, TG, TV, TC, true, DIR == 3 || (DIR == 0 && STREAM), false, NTG,
          DIR != 0, false, DIR, true>(
      threadIdx.x, e0, sd.E, D, G, u, w, &sd.box, smem, nullptr, DIR ? sd.edot : nullptr,
      DIR == 1 || DIR == 2 ? &dir : nullptr);
}

template <int BS, class TV, class TG, class TC, int DIR, bool STREAM, int... N1s>
__global__ void __launch_bounds__(BS)
    k_bax(const BatchSolve *__restrict__ sds, CgState *st,
          const AxItem *__restrict__ items, int nitems, int src, BaxDir bd) {
  extern __shared__ __align__(16) unsigned char dyn_smem[];
  TC *smem = reinterpret_cast<TC *>(dyn_smem);
  // a workgroup walks a run of consecutive items, and the workgroups of an
  // XCD take consecutive runs: their elements share nodes of the gathered
  // vector.  The next item is asked for before the current one's work, so
  // that its latency is hidden
  const int run = (nitems + (int)gridDim.x - 1) / (int)gridDim.x;
  const int q0 = (int)xcd_run_block(blockIdx.x, gridDim.x) * run;
  const int q1 = min(q0 + run, nitems);
  AxItem next = q0 < q1 ? items[q0] : AxItem{};
  for (int q = q0; q < q1; ++q) {
    const AxItem it = next;
    if (q + 1 < q1) next = items[q + 1];
    const BatchSolve &sd = sds[it.solve];
    DirArgs<TV> dir = {};
    if constexpr (DIR == 1 || DIR == 2) dir = batch_dir<TV>(sd, st, bd, it.solve);
    // a finished solve: at most its first tile goes on, to pass the flag to
    // the r update
    if (DIR != 0 && st[it.solve].done != 0 && (DIR == 3 || it.elem0 != 0))
      continue;  // uniform per block
    const int n1 = sd.N1;
    // exactly one of the compiled orders matches the item's order
    ((n1 == N1s ? bax_one<BS, TV, TG, TC, DIR, STREAM, N1s>(sd, it.elem0, src, dir, smem)
                : void()),
     ...);
    __syncthreads();  // the next item may use another LDS layout
  }
}

template <int BS, class TC, int... N1s> constexpr int max_lds_words() {
  int m = 0;
  ((m = lds_words<N1s, TC>(BTile<BS, N1s>::EPB) > m
            ? lds_words<N1s, TC>(BTile<BS, N1s>::EPB)
            : m),
   ...);
  return m;
}

template <int BS, class TV, class TG, class TC, int DIR, bool STREAM, int... N1s>
static void launch_bax_set(const BatchSolve *sds, CgState *st, const AxItem *items,
                           int nitems, int grid, int src, const BaxDir &bd,
                           hipStream_t s) {
  const size_t lds = (size_t)max_lds_words<BS, TC, N1s...>() * sizeof(TC);
  hipLaunchKernelGGL((k_bax<BS, TV, TG, TC, DIR, STREAM, N1s...>), dim3(grid), dim3(BS), lds,
                     s, sds, st, items, nitems, src, bd);
}

template <int BS, class TV, class TG, class TC, int DIR, bool STREAM>
static void launch_bax_bs(int nset, const BatchSolve *sds, CgState *st,
                          const AxItem *items, int nitems, int grid, int src,
                          const BaxDir &bd, hipStream_t s) {
  // a thread owns one (i, j) column: a workgroup must hold every column of
  // the largest order of the set
  if (BS < bax_min_block(nset))
    fail(SEM_ERR_ARG, "batched operator: block size below n1^2 of an order");
  // order sets compiled: one order (n1 = 2..9) or the mixed set {4, 6, 8}
  switch (nset) {
#define SEM_BAX_SET(...)                                                                  \
  launch_bax_set<BS, TV, TG, TC, DIR, STREAM, __VA_ARGS__>(sds, st, items, nitems, grid, src, \
                                                           bd, s)
#define SEM_BAX(...)        \
  SEM_BAX_SET(__VA_ARGS__); \
  break
    case 2: SEM_BAX(2);
    case 3: SEM_BAX(3);
    case 4: SEM_BAX(4);
    case 5: SEM_BAX(5);
    case 6: SEM_BAX(6);
    case 7: SEM_BAX(7);
    case 8: SEM_BAX(8);
    case 9:
      if constexpr (BS >= 81) SEM_BAX_SET(9);  // (smaller blocks are refused above)
      break;
    case AX_SET_468: SEM_BAX(4, 6, 8);
#undef SEM_BAX
#undef SEM_BAX_SET
    default: fail(SEM_ERR_ARG, "batched operator: unsupported set of orders");
  }
}

template <class TV, class TG, class TC, int DIR, bool STREAM>
static void launch_bax_t(int bs, int nset, const BatchSolve *sds, CgState *st,
                         const AxItem *items, int nitems, int grid, int src,
                         const BaxDir &bd, hipStream_t s) {
  switch (bs) {
    case 64: launch_bax_bs<64, TV, TG, TC, DIR, STREAM>(nset, sds, st, items, nitems, grid, src, bd, s); break;
    case 128: launch_bax_bs<128, TV, TG, TC, DIR, STREAM>(nset, sds, st, items, nitems, grid, src, bd, s); break;
    case 256: launch_bax_bs<256, TV, TG, TC, DIR, STREAM>(nset, sds, st, items, nitems, grid, src, bd, s); break;
    default: fail(SEM_ERR_ARG, "batched operator: block size must be 64, 128 or 256");
  }
}

template <int DIR, bool STREAM>
static void launch_bax_d(int prec, int bs, int nset, const BatchSolve *sds, CgState *st,
                         const AxItem *items, int nitems, int grid, int src,
                         const BaxDir &bd, hipStream_t s) {
  if (prec == SEM_FP64)
    launch_bax_t<double, double, double, DIR, STREAM>(bs, nset, sds, st, items, nitems, grid, src,
                                              bd, s);
  else if (prec == SEM_FP32)
    launch_bax_t<float, float, float, DIR, STREAM>(bs, nset, sds, st, items, nitems, grid, src, bd,
                                           s);
  else
    launch_bax_t<float, uint16_t, float, DIR, STREAM>(bs, nset, sds, st, items, nitems, grid, src,
                                              bd, s);
}

void launch_bax(int prec, int bs, int nset, const BatchSolve *sds, CgState *st,
                const AxItem *items, int nitems, int grid, int src, const BaxDir &bd,
                hipStream_t s) {
  if (nitems <= 0) return;
  if (bd.mode == 0) {
    // the residuals: FP64
    if (prec != SEM_FP64) fail(SEM_ERR_ARG, "batched operator: FP64 outside an iteration");
    auto go = bd.stream ? launch_bax_t<double, double, double, 0, true>
                        : launch_bax_t<double, double, double, 0, false>;
    go(bs, nset, sds, st, items, nitems, grid, src, bd, s);
  } else if (bd.mode == 1)
    bd.stream ? launch_bax_d<1, true>(prec, bs, nset, sds, st, items, nitems, grid, src, bd, s)
              : launch_bax_d<1, false>(prec, bs, nset, sds, st, items, nitems, grid, src, bd, s);
  else if (bd.mode == 2)
    launch_bax_d<2, false>(prec, bs, nset, sds, st, items, nitems, grid, src, bd, s);
  else
    launch_bax_d<3, true>(prec, bs, nset, sds, st, items, nitems, grid, src, bd, s);
  SEM_HIP(hipGetLastError());
}

int bax_min_block(int nset) {
  const int n1 = nset == AX_SET_468 ? 8 : nset;
  const int np = n1 * n1;
  return np <= 64 ? 64 : np <= 128 ? 128 : 256;
}

int bax_elements_per_tile(int bs, int n1) {
  const int np = n1 * n1;
  return bs / np > 0 ? bs / np : 1;
}

}  // namespace sem
