"""The flexible CG's dot products with the coarse correction, summed a term
per workgroup of four elements: element counts around whole workgroups,
against the oracle's flexible CG with the same preconditioner."""
import numpy as np
import pytest

from oracle import oracle as orc
from seminputs import fourier_modes

from gpu_util import Pair, to_dev, to_host, torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,box", [(2, (5, 1, 1)), (3, (3, 1, 1)), (4, (2, 2, 1)), (7, (1, 1, 1)),
                                   (5, (5, 13, 1)), (7, (3, 3, 7)), (3, (17, 4, 16))])
def test_iterates(N, box):
    """x after 5 iterations: the correction is rounded to FP32 (6e-8), which
    5 iterations amplify by far less than 100, while one lost or doubled
    element term changes beta by at least 1e-4 of itself."""
    from paper_1403_0968_amd import sem
    print(f"[gpu] fcg terms N={N} {box}", flush=True)
    t = torch()
    pr = Pair(sem, N, *box, mapping=sem.SEM_MAP_SINE_CYCLIC)
    m = pr.m
    try:
        sem.sem_learn_attach_exact(pr.h, 1.0)
        b = t.empty(pr.nL, dtype=t.float64, device="cuda")
        sem.sem_rhs(pr.h, b, sem.SEM_SRC_FOURIER, fourier_modes(seed=3))
        x = t.zeros_like(b)
        st = sem.sem_pcg_solve(pr.h, b, x, rtol=1e-13, maxit=5, check_every=4,
                               pc=sem.SEM_PC_LEARNED, raise_on_fail=False)
        t.cuda.synchronize()

        def prec(r):
            rl = to_dev(orc.to_local(m, r))
            z = t.empty_like(rl)
            sem.sem_precond_apply(pr.h, sem.SEM_PC_LEARNED, sem.SEM_FP64, rl, z)
            return orc.to_global(m, to_host(z))

        xo, _, its, _ = orc.fcg(m, orc.to_global(m, to_host(b)), prec, 1e-13, 5)
        xo = orc.to_local(m, xo)
        err = np.linalg.norm(to_host(x) - xo) / np.linalg.norm(xo)
        print(f"[fcg] its {st['iters']} {its} err {err:.2e}")
        assert st["iters"] == its
        assert err <= 6e-6, err
    finally:
        t.cuda.synchronize()
        pr.close()
