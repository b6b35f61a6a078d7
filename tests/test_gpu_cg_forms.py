"""The forms of the CG iteration against each other and the oracle.

Small solves add the partial sums inside the operator and the r update and
form the search direction at the operator's gather; larger ones run scalar
kernels for the sums; vectors beyond the last-level cache get a pass of
their own for p and x.  Which form runs depends on the sizes of all solves
of a call, and every form must give the same bits: a small solve is run
alone and beside partners that move the whole batch to the other forms, at
even and odd numbers of iterations per launch sequence (the two direction
buffers swap roles at each iteration)."""
import numpy as np
import pytest

from oracle import oracle as orc
from seminputs import fourier_modes

from gpu_util import Pair, to_host, torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sem():
    from paper_1403_0968_amd import sem as s
    s.lib()
    return s


def _rhs(sem, h, seed):
    t = torch()
    b = t.empty(sem.sem_query(h)[1], dtype=t.float64, device="cuda")
    sem.sem_rhs(h, b, sem.SEM_SRC_FOURIER, fourier_modes(seed=seed))
    return b


def _side(N, n_local):
    return round((n_local / (N + 1) ** 3) ** (1 / 3))


# (N, box, periodic): one element, ragged boxes, both copies of a periodic
# direction in one element, a last chunk of a few nodes
SMALL = [(1, (5, 3, 4), 0, "fp64 fp32 bf16_mfma"), (2, (1, 1, 1), 0, "fp64"),
         (3, (4, 2, 3), 0, "fp64 bf16"), (4, (3, 4, 5), 3, "fp64 fp32"),
         (5, (2, 1, 3), 2, "fp64"), (6, (3, 2, 2), 0, "fp32 bf16_mfma"),
         (7, (5, 4, 3), 0, "fp64 fp32 bf16 bf16_mfma"),
         (8, (2, 3, 2), 5, "fp64 fp32 bf16_mfma")]


@pytest.mark.parametrize("N,box,per,prec", [(N, box, per, p) for N, box, per, ps in SMALL
                                            for p in ps.split()])
def test_forms_give_the_same_bits(sem, N, box, per, prec):
    print(f"[gpu] cg forms N={N} {box} periodic={per} {prec}", flush=True)
    t = torch()
    p = {"fp64": sem.SEM_FP64, "fp32": sem.SEM_FP32, "bf16": sem.SEM_BF16,
         "bf16_mfma": sem.SEM_BF16_MFMA}[prec]
    value = 8 if prec == "fp64" else 4
    # beyond RED_ENERGIES elements or RED_PARTS chunks; vectors beyond 128 MiB
    # (about 5 unique-node vectors and the E-vector)
    mid = _side(N, 1.3e6)
    big = _side(N, 1.3 * 128 * 2 ** 20 / value / (1 + 5 * (N / (N + 1)) ** 3))
    hs = [sem.sem_setup(N, *box, mapping=sem.SEM_MAP_SINE_CYCLIC, periodic=per)]
    hs += [sem.sem_setup(N, n, n, n) for n in (mid, big)]
    try:
        _, nL, nG = sem.sem_query(hs[2])
        assert value * (5 * nG + nL) > 128 * 2 ** 20
        _, nL, nG = sem.sem_query(hs[1])
        assert value * (5 * nG + nL) < 120 * 2 ** 20
        bs = [_rhs(sem, h, 7 + q) for q, h in enumerate(hs)]
        kw = dict(rtol=1e-9, maxit=37, inner_prec=p, inner_rtol=1e-2,
                  raise_on_fail=False)
        xs, its = [], []
        for every, graph in ((4, 1), (3, 1), (1, 0), (5, 0)):
            x = t.zeros_like(bs[0])
            its.append(sem.sem_pcg_solve(hs[0], bs[0], x, check_every=every,
                                         use_graph=graph, **kw)["iters"])
            xs.append(x)
        # (at N = 1 the batched and the single matrix-core refinement differ in
        # the last bits, whatever the form)
        for q, every in ((1, 4), (2, 4), (1, 3), (2, 3)) if (N, prec) != (1, "bf16_mfma") else ():
            bt = sem.sem_batch_create([hs[0], hs[q]])
            x = [t.zeros_like(bs[0]), t.zeros_like(bs[q])]
            _, st = sem.sem_batch_pcg_solve(bt, [bs[0], bs[q]], x, check_every=every, **kw)
            t.cuda.synchronize()
            sem.sem_batch_destroy(bt)
            its.append(st[0]["iters"])
            xs.append(x[0])
        t.cuda.synchronize()
        assert len(set(its)) == 1, its
        scale = xs[0].abs().max()
        off = [float((x - xs[0]).abs().max() / scale) for x in xs]
        assert off == [0.0] * len(xs), off
        assert bool(xs[0].abs().max() > 0)
    finally:
        t.cuda.synchronize()
        for h in hs:
            sem.sem_destroy(h)


# element counts and chunk counts on both sides of the limits for adding the
# sums in the two passes (4096 energies, 1024 chunks of 1024 nodes)
@pytest.mark.parametrize("N,box", [(1, (16, 16, 16)), (1, (17, 121, 2)), (2, (63, 64, 65)),
                                   (2, (64, 64, 63)), (7, (6, 7, 9)), (4, (12, 11, 10))])
def test_limits_match_oracle_iterates(sem, N, box):
    """x after 6 iterations against the oracle's PCG: 6 iterations of CG
    amplify the rounding of the operator (1e-12 relative at most) by far less
    than 1e4, so 1e-8 separates rounding from a lost or doubled term."""
    print(f"[gpu] cg limits N={N} {box}", flush=True)
    t = torch()
    pr = Pair(sem, N, *box, mapping=sem.SEM_MAP_SINE_CYCLIC)
    b = _rhs(sem, pr.h, 3)
    x = t.zeros_like(b)
    st = sem.sem_pcg_solve(pr.h, b, x, rtol=1e-14, maxit=6, check_every=4,
                           raise_on_fail=False)
    t.cuda.synchronize()
    assert st["iters"] == 6
    bo = orc.to_global(pr.m, to_host(b))
    xo = orc.to_local(pr.m, orc.pcg(pr.m, bo, 1e-14, 6)[0])
    err = np.linalg.norm(to_host(x) - xo) / np.linalg.norm(xo)
    assert err <= 1e-8, err
    pr.close()


# a mesh of its own size class alone (the single-solve operator in the shapes
# for meshes in and beyond the caches) against the batched operator beside a
# small partner: the same bits
@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("N", range(1, 9))
def test_single_shapes_equal_batched(sem, N, prec):
    print(f"[gpu] single against batch N={N} {prec}", flush=True)
    t = torch()
    p = {"fp64": sem.SEM_FP64, "fp32": sem.SEM_FP32, "bf16": sem.SEM_BF16}[prec]
    value = 8 if prec == "fp64" else 4
    per_node = value * (1 + 5 * (N / (N + 1)) ** 3)  # vectors, bytes per local node
    small = sem.sem_setup(N, 2, 2, 3)
    try:
        # 0.9M nodes (in the caches; ragged so that the last workgroup is
        # partial), and vectors beyond 128 MiB
        n = _side(N, 0.9e6)
        big = _side(N, 1.2 * 128 * 2 ** 20 / per_node)
        for box in ((n, n + 1, n), (big, big, big + 1)):
            h = sem.sem_setup(N, *box, mapping=sem.SEM_MAP_SINE_CYCLIC)
            b, b0 = _rhs(sem, h, 3), _rhs(sem, small, 4)
            kw = dict(rtol=1e-9, maxit=5, inner_prec=p, inner_rtol=1e-2, check_every=4,
                      raise_on_fail=False)
            x = t.zeros_like(b)
            sem.sem_pcg_solve(h, b, x, **kw)
            bt = sem.sem_batch_create([small, h])
            xs = [t.zeros_like(b0), t.zeros_like(b)]
            sem.sem_batch_pcg_solve(bt, [b0, b], xs, **kw)
            t.cuda.synchronize()
            sem.sem_batch_destroy(bt)
            off = float((x - xs[1]).abs().max() / x.abs().max())
            sem.sem_destroy(h)
            assert off == 0.0, (box, off)
    finally:
        sem.sem_destroy(small)
