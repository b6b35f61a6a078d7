"""The standalone operator at N = 7 on either side of the lines between which
its streaming forms run inside the last-level cache (38 and 130 MiB moved per
application: 64, 32 or 18 bytes a node, with a mass term 72, 36 or 20),
against plain FP64 products of the exported factors.  Tolerances: sums of 24
products each way, FP64 1e-12, FP32 arithmetic 2e-6 of the largest entry."""
import numpy as np
import pytest

from oracle import oracle as orc

from gpu_util import torch
from test_gpu_ax_shapes import _reference

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("above", [0, 1])
@pytest.mark.parametrize("mib", [38, 130])
@pytest.mark.parametrize("alpha", [0.0, 2.0])
@pytest.mark.parametrize("prec,per", [("fp64", (64, 72)), ("fp32", (32, 36)), ("bf16", (18, 20))])
def test_operator_at_the_lines(prec, per, alpha, mib, above):
    from paper_1403_0968_amd import sem
    t = torch()
    per = per[1] if alpha else per[0]
    ez = int(mib * 2 ** 20 / (per * 512 * 121)) + above
    print(f"[gpu] ax band {prec} alpha={alpha} 11x11x{ez}", flush=True)
    h = sem.sem_setup(7, 11, 11, ez, mapping=sem.SEM_MAP_SINE_CYCLIC, alpha=alpha)
    try:
        E, nL, _ = sem.sem_query(h)
        assert (nL * per > mib * 2 ** 20) == bool(above)
        g = t.Generator(device="cuda")
        g.manual_seed(mib)
        u = t.rand(nL, dtype=t.float64, device="cuda", generator=g) * 2 - 1
        G = t.empty(6 * nL, dtype=t.float64, device="cuda")
        sem.sem_export(h, sem.SEM_ARR_GEOM, G)
        H = t.zeros(nL, dtype=t.float64, device="cuda")
        if alpha:
            sem.sem_export(h, sem.SEM_ARR_HMASS, H)
        dt = {"fp64": t.float64, "fp32": t.float32, "bf16": t.bfloat16}[prec]
        ui = u.to(dt)
        u, G, H = ui.double(), G.to(dt).double(), H.to(dt).double()
        w = t.full((nL + 1,), 7.0, dtype=t.float64 if prec == "fp64" else t.float32,
                   device="cuda")
        p = {"fp64": sem.SEM_FP64, "fp32": sem.SEM_FP32, "bf16": sem.SEM_BF16}[prec]
        for _ in range(2):
            sem.sem_ax(h, p, ui, w)
        t.cuda.synchronize()
        D = t.as_tensor(np.asarray(orc.dmat(7, orc.gll(7)[0])), device="cuda")
        ref = _reference(G, D, u.view(E, 8, 8, 8)).reshape(-1) + H * u
        err = float((w[:nL].double() - ref).abs().max() / ref.abs().max())
        assert float(w[nL]) == 7.0
        assert err <= (1e-12 if prec == "fp64" else 2e-6), err
    finally:
        t.cuda.synchronize()
        sem.sem_destroy(h)
