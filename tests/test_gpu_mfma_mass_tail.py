"""Matrix-core refinement of the screened operator (section 4.2, equation
semPDE with alpha != 0) where the last workgroup of the operator is partial:
every order at element counts that leave waves without an element (four
elements per workgroup, two at N = 8).  Those waves read no mass factor.
The solution to 1e-10 against the FP64 solve's: both residuals are below
1e-10 and the condition numbers of these meshes below 1e3, so 1e-6."""
import pytest

from seminputs import fourier_modes

from gpu_util import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,box", [(1, (5, 3, 3)), (2, (3, 3, 1)), (3, (3, 2, 1)),
                                   (4, (1, 3, 1)), (5, (2, 3, 1)), (6, (3, 1, 1)),
                                   (7, (1, 1, 1)), (8, (3, 1, 1))])
def test_partial_workgroup_with_mass(N, box):
    from paper_1403_0968_amd import sem
    print(f"[gpu] matrix-core solve with mass N={N} {box}", flush=True)
    t = torch()
    h = sem.sem_setup(N, *box, mapping=sem.SEM_MAP_SINE_CYCLIC, dirichlet=0, alpha=2.0)
    try:
        b = t.empty(sem.sem_query(h)[1], dtype=t.float64, device="cuda")
        sem.sem_rhs(h, b, sem.SEM_SRC_FOURIER, fourier_modes(seed=N))
        xs = []
        for prec in (sem.SEM_FP64, sem.SEM_BF16_MFMA):
            x = t.zeros_like(b)
            st = sem.sem_pcg_solve(h, b, x, rtol=1e-10, maxit=5000, inner_prec=prec,
                                   check_every=8)
            assert st["status"] == 0 and st["final_rel_res"] <= 1e-10
            xs.append(x)
        t.cuda.synchronize()
        assert float((xs[1] - xs[0]).norm() / xs[0].norm()) <= 1e-6
    finally:
        sem.sem_destroy(h)
