"""Matrix-core operators on more elements than one launch has threads for (a
wave of 64 each, 2^32 threads a launch): N = 1, 407^3 elements, 84 GB.
The standalone operator at elements within and at the end against plain FP64
products of their BF16 factors (fluxes rounded to BF16: 2e-2), with one value
past the end kept; the refinement's operator against the one of a batch, whose
workgroups take 64 elements each and fit one launch: a solve gives the same
bits alone and beside another."""
import numpy as np
import pytest

from oracle import oracle as orc

from gpu_util import torch
from test_gpu_ax_shapes import _reference

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mesh():
    from paper_1403_0968_amd import sem
    t = torch()
    print("[gpu] N=1 407^3", flush=True)
    h = sem.sem_setup(1, 407, 407, 407)
    yield h
    t.cuda.synchronize()
    sem.sem_destroy(h)
    t.cuda.empty_cache()


def test_operator(mesh):
    from paper_1403_0968_amd import sem
    t = torch()
    E, nL, _ = sem.sem_query(mesh)
    assert 64 * E > 1 << 32
    G = t.empty(6 * nL, dtype=t.float64, device="cuda")
    sem.sem_export(mesh, sem.SEM_ARR_GEOM, G)
    places = t.tensor([0, (1 << 25) - 1, 1 << 25, E // 3, 1 << 26, E - 1], device="cuda")
    G = G.view(E, 48)[places].contiguous()
    g = t.Generator(device="cuda")
    g.manual_seed(1)
    u = (t.rand(nL, device="cuda", generator=g) - 0.5).bfloat16()
    w = t.full((nL + 1,), 7.0, device="cuda")
    sem.sem_ax(mesh, sem.SEM_BF16_MFMA, u, w)
    t.cuda.synchronize()
    D = t.as_tensor(np.asarray(orc.dmat(1, orc.gll(1)[0])), device="cuda")
    x = u.view(E, 8)[places].double().view(-1, 2, 2, 2).contiguous()
    ref = _reference(G.bfloat16().double(), D, x).reshape(-1, 8)
    got = w[:nL].view(E, 8)[places].double()
    err = (got - ref).abs().amax(1) / ref.abs().amax(1)
    assert float(err.max()) <= 2e-2, err
    assert float(w[nL]) == 7.0


def test_refinement(mesh):
    from paper_1403_0968_amd import sem
    t = torch()
    nL = sem.sem_query(mesh)[1]
    b = t.empty(nL, dtype=t.float64, device="cuda")
    k = np.array([[1.0, 2.0, 1.0], [40.0, 33.0, 57.0]])
    sem.sem_rhs(mesh, b, sem.SEM_SRC_FOURIER, (k, np.array([1.0, 30.0]), np.array([0.3, 1.1])))
    small = sem.sem_setup(1, 3, 3, 3)
    b2 = t.empty(sem.sem_query(small)[1], dtype=t.float64, device="cuda")
    sem.sem_rhs(small, b2, sem.SEM_SRC_FOURIER, (k, np.array([1.0, 30.0]), np.array([0.3, 1.1])))
    kw = dict(rtol=1e-9, maxit=3, inner_prec=sem.SEM_BF16_MFMA, inner_rtol=1e-3,
              check_every=3, raise_on_fail=False)
    x = t.zeros_like(b)
    assert sem.sem_pcg_solve(mesh, b, x, **kw)["iters"] == 3
    bt = sem.sem_batch_create([small, mesh])
    try:
        xs = [t.zeros_like(b2), t.zeros_like(b)]
        sem.sem_batch_pcg_solve(bt, [b2, b], xs, **kw)
        t.cuda.synchronize()
        assert float(x[-nL // 10:].abs().max()) > 0.05 * float(x.abs().max()) > 0
        assert t.equal(x, xs[1])
    finally:
        sem.sem_batch_destroy(bt)
        sem.sem_destroy(small)
