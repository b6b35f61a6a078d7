"""Matrix-core refinement: a solve gives the bits of the same solve run alone
inside any batch, at every order and for both forms of the derivative matrix
(include/sem.h, batches of independent solves).  The partners leave the batch
in the form of two passes (a small one) and move it to the form with a pass of
its own for p and x (vectors beyond 128 MiB, orders 1 and 2, where the
compiler once contracted the direction's update differently in the two
kernels); 2, 3 and 12 iterations, so that a difference in one direction shows
before the refinement hides it."""
import pytest

from seminputs import fourier_modes

from gpu_util import torch

pytestmark = pytest.mark.gpu


def _rhs(sem, h, seed):
    t = torch()
    b = t.empty(sem.sem_query(h)[1], dtype=t.float64, device="cuda")
    sem.sem_rhs(h, b, sem.SEM_SRC_FOURIER, fourier_modes(seed=seed))
    return b


@pytest.mark.parametrize("plain", [0, 1])
@pytest.mark.parametrize("N", range(1, 9))
def test_alone_equals_batch(N, plain):
    from paper_1403_0968_amd import sem
    print(f"[gpu] matrix-core bits N={N} plain={plain}", flush=True)
    t = torch()
    prec = sem.SEM_BF16_PLAIN_D if plain else sem.SEM_BF16_MFMA
    boxes = [(5, 3, 4), (2, 2, 3)]
    if N <= 2 and not plain:
        side = round((1.3 * 2 ** 25 / (1 + 5 * (N / (N + 1)) ** 3)) ** (1 / 3) / (N + 1))
        boxes.append((side, side, side))
    hs = [sem.sem_setup(N, *box, mapping=sem.SEM_MAP_SINE_CYCLIC) for box in boxes]
    try:
        bs = [_rhs(sem, h, 3 + q) for q, h in enumerate(hs)]
        if len(hs) == 3:
            _, nL, nG = sem.sem_query(hs[2])
            assert 4 * (5 * nG + nL) > 128 * 2 ** 20
        for maxit in (2, 3, 12):
            kw = dict(rtol=1e-9, maxit=maxit, inner_prec=prec, inner_rtol=1e-2,
                      check_every=4, raise_on_fail=False)
            x = t.zeros_like(bs[0])
            sem.sem_pcg_solve(hs[0], bs[0], x, **kw)
            t.cuda.synchronize()
            assert bool(x.abs().max() > 0)
            for q in range(1, len(hs)):
                bt = sem.sem_batch_create([hs[0], hs[q]])
                xs = [t.zeros_like(bs[0]), t.zeros_like(bs[q])]
                sem.sem_batch_pcg_solve(bt, [bs[0], bs[q]], xs, **kw)
                t.cuda.synchronize()
                sem.sem_batch_destroy(bt)
                assert t.equal(x, xs[0]), (maxit, boxes[q])
    finally:
        t.cuda.synchronize()
        for h in hs:
            sem.sem_destroy(h)
