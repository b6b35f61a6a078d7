"""The standalone operator in the workgroup shapes and load hints of every
size class (at most 0.2M local nodes, in the last-level cache, beyond it),
element counts that leave the last workgroup partial, against plain FP64
products of the exported factors.

Tolerances: sums of 3 (N+1) products each way; FP64 1e-12, FP32 2e-6 of the
largest entry, BF16 operands with FP32 arithmetic 2e-6 against the same
rounded operands, the matrix-core operator 2e-2 (fluxes rounded to BF16)."""
import numpy as np
import pytest

from oracle import oracle as orc

from gpu_util import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sem():
    from paper_1403_0968_amd import sem as s
    s.lib()
    return s


def _reference(G, D, u):
    """w = D^T G D u in FP64; G [E][6][n1^3], u [E][k][j][i]."""
    t = torch()
    E, n1 = u.shape[0], u.shape[1]
    g = G.view(E, 6, n1, n1, n1)
    DT = D.T.contiguous()
    ur = (u.reshape(-1, n1) @ DT).view(u.shape)
    us = t.matmul(D, u)
    ut = t.matmul(D, u.reshape(E, n1, -1)).view(u.shape)
    w = ((g[:, 0] * ur + g[:, 1] * us + g[:, 2] * ut).reshape(-1, n1) @ D).view(u.shape)
    w += t.matmul(DT, g[:, 1] * ur + g[:, 3] * us + g[:, 4] * ut)
    f = g[:, 2] * ur + g[:, 4] * us + g[:, 5] * ut
    w += t.matmul(DT, f.reshape(E, n1, -1)).view(u.shape)
    return w


# local nodes of the size classes by precision (bytes per node 64, 32, 18;
# 256 MiB): just above 0.2M, and beyond the cache
SIZES = [(N, prec, nodes)
         for N in range(1, 9)
         for prec, nodes in [("fp64", 2.1e5), ("fp32", 2.1e5), ("bf16", 2.1e5),
                             ("bf16_mfma", 2.1e5), ("fp64", 5.4e6)]]
SIZES += [(N, "fp32", 1.07e7) for N in (2, 3, 5, 6, 7, 8)]
SIZES += [(N, "bf16", 1.9e7) for N in (1, 4, 7)] + [(7, "bf16_mfma", 1.9e7)]


@pytest.mark.parametrize("N,prec,nodes", SIZES)
def test_operator(sem, N, prec, nodes):
    print(f"[gpu] ax shapes N={N} {prec} {nodes:.3g} nodes", flush=True)
    t = torch()
    n1 = N + 1
    n = round((nodes / n1 ** 3) ** (1 / 3))
    ez = max(1, int(np.ceil(nodes / (n1 ** 3 * n * n))))
    h = sem.sem_setup(N, n, n, ez, mapping=sem.SEM_MAP_SINE_CYCLIC)
    try:
        E, nL, _ = sem.sem_query(h)
        assert nL >= nodes
        g = t.Generator(device="cuda")
        g.manual_seed(N)
        u = t.rand(nL, dtype=t.float64, device="cuda", generator=g) * 2 - 1
        G = t.empty(6 * nL, dtype=t.float64, device="cuda")
        sem.sem_export(h, sem.SEM_ARR_GEOM, G)
        out = t.float64 if prec == "fp64" else t.float32
        # one value past the end must stay
        w = t.full((nL + 1,), 7.0, dtype=out, device="cuda")
        if prec == "fp64":
            ui = u
        elif prec == "fp32":
            ui = u.float()
            u, G = ui.double(), G.float().double()
        else:
            b = u.bfloat16()
            ui = b.view(t.int16)
            u, G = b.double(), G.bfloat16().double()
        p = {"fp64": sem.SEM_FP64, "fp32": sem.SEM_FP32, "bf16": sem.SEM_BF16,
             "bf16_mfma": sem.SEM_BF16_MFMA}[prec]
        for _ in range(2):
            sem.sem_ax(h, p, ui, w)
        t.cuda.synchronize()
        D = t.as_tensor(orc.dmat(N, orc.gll(N)[0]), device="cuda")
        ref = _reference(G, D, u.view(E, n1, n1, n1)).reshape(-1)
        err = float((w[:nL].double() - ref).abs().max() / ref.abs().max())
        print(f"[ax] {err:.2e}")
        assert float(w[nL]) == 7.0
        assert err <= {"fp64": 1e-12, "fp32": 2e-6, "bf16": 2e-6, "bf16_mfma": 2e-2}[prec]
    finally:
        t.cuda.synchronize()
        sem.sem_destroy(h)
