"""The sum of the element energies of meshes of many elements (in chunks of
8192 beyond 32768): element counts around whole chunks, a periodic mesh with
as many unique nodes as elements, and solves of both kinds in one batch."""
import numpy as np
import pytest

from oracle import oracle as orc
from seminputs import fourier_modes

from gpu_util import Pair, to_host, torch

pytestmark = pytest.mark.gpu


def _rhs(sem, h):
    t = torch()
    b = t.empty(sem.sem_query(h)[1], dtype=t.float64, device="cuda")
    sem.sem_rhs(h, b, sem.SEM_SRC_FOURIER, fourier_modes(seed=3))
    return b


@pytest.mark.parametrize("box,per", [((32, 32, 32), 0), ((9, 11, 331), 0), ((11, 43, 70), 0),
                                     ((64, 64, 9), 0), ((16, 16, 160), 0), ((33, 32, 32), 7)])
def test_iterates_and_batch(box, per):
    """x after 6 iterations against the oracle's PCG (6 iterations amplify
    the rounding of the operator, 1e-12 at most, by far less than 1e4), and
    the same bits in a batch with a small solve."""
    from paper_1403_0968_amd import sem
    print(f"[gpu] energies {box} per={per}", flush=True)
    t = torch()
    pr = Pair(sem, 1, *box, mapping=sem.SEM_MAP_SINE_CYCLIC, periodic=per,
              alpha=1.0 if per else 0.0)
    small = sem.sem_setup(1, 4, 3, 5)
    try:
        b, b0 = _rhs(sem, pr.h), _rhs(sem, small)
        kw = dict(rtol=1e-14, maxit=6, check_every=4, raise_on_fail=False)
        x, xs = t.zeros_like(b), [t.zeros_like(b0), t.zeros_like(b)]
        sem.sem_pcg_solve(pr.h, b, x, **kw)
        if not per:  # (a mass term is solved singly)
            bt = sem.sem_batch_create([small, pr.h])
            sem.sem_batch_pcg_solve(bt, [b0, b], xs, **kw)
            t.cuda.synchronize()
            sem.sem_batch_destroy(bt)
            assert t.equal(x, xs[1])
        xo = orc.to_local(pr.m, orc.pcg(pr.m, orc.to_global(pr.m, to_host(b)), 1e-14, 6)[0])
        err = np.linalg.norm(to_host(x) - xo) / np.linalg.norm(xo)
        assert err <= 1e-8, err
    finally:
        t.cuda.synchronize()
        sem.sem_destroy(small)
        pr.close()
