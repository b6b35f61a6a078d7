"""Coarse correction on 2^24 elements and more (N = 2, 256 x 256 x 257, 69 GB):
the operators M_e of every element are filled, from a network and exactly.
On an affine mesh with constant coefficient they are alike, and a constant
residual gives the same bits in every element's interior node."""
import numpy as np
import pytest

from gpu_util import torch

pytestmark = pytest.mark.gpu


def test_operators_of_every_element():
    from paper_1403_0968_amd import sem
    t = torch()
    print("[gpu] coarse correction N=2 256x256x257", flush=True)
    h = sem.sem_setup(2, 256, 256, 257)
    net = sem.sem_mlp_create(8, 128, 1, seed=1)  # (its output layer starts at zero)
    n = sem.sem_mlp_info(net)["n_params"]
    sem.sem_mlp_set_params(net, np.random.default_rng(1).normal(0.0, 0.2, n))
    try:
        E, nL, _ = sem.sem_query(h)
        assert 256 * E > 1 << 32
        r = t.ones(nL, dtype=t.float64, device="cuda")
        for exact in (0, 1):
            if exact:
                sem.sem_learn_attach_exact(h, 1.0)
            else:
                sem.sem_learn_attach(h, net)
            z = t.full((nL,), 7.0, dtype=t.float64, device="cuda")
            sem.sem_precond_apply(h, sem.SEM_PC_JACOBI, sem.SEM_FP64, r, z)
            j = z.view(E, 27)[:, 13].clone()
            sem.sem_precond_apply(h, sem.SEM_PC_LEARNED, sem.SEM_FP64, r, z)
            t.cuda.synchronize()
            c = z.view(E, 27)[:, 13] - j
            first = float(c[0])
            assert first != 0.0
            # the Jacobi part differs by the rounding of the coordinates
            assert float((c - first).abs().max()) <= 1e-5 * abs(first)
            del z, j, c
    finally:
        t.cuda.synchronize()
        sem.sem_learn_attach(h, None)
        sem.sem_mlp_destroy(net)
        sem.sem_destroy(h)
        t.cuda.empty_cache()
