"""A mesh of more than 2^32 geometric factors (N = 7, 112^3 elements, 719M
nodes, 108 GB of the card): every element has its FP32 and BF16 factors.
Elements at the start, within and at the end against plain FP64 products of
their exported factors rounded to the precision (FP32 arithmetic, sums of 24
products each way: 2e-6 of the largest entry)."""
import numpy as np
import pytest

from oracle import oracle as orc

from gpu_util import torch
from test_gpu_ax_shapes import _reference

pytestmark = pytest.mark.gpu


def test_factors_of_every_element():
    from paper_1403_0968_amd import sem
    t = torch()
    print("[gpu] large mesh N=7 112^3", flush=True)
    h = sem.sem_setup(7, 112, 112, 112)
    try:
        E, nL, _ = sem.sem_query(h)
        assert 6 * nL > 1 << 32
        places = (0, E // 3, E // 2, E - 1)
        G = t.empty(6 * nL, dtype=t.float64, device="cuda")
        sem.sem_export(h, sem.SEM_ARR_GEOM, G)
        G = t.stack([G[3072 * e:3072 * (e + 1)] for e in places])
        D = t.as_tensor(np.asarray(orc.dmat(7, orc.gll(7)[0])), device="cuda")
        g = t.Generator(device="cuda")
        g.manual_seed(7)
        v = t.rand(512, device="cuda", generator=g) - 0.5
        for p, dt in ((sem.SEM_FP32, t.float32), (sem.SEM_BF16, t.bfloat16)):
            u = t.zeros(nL, dtype=dt, device="cuda")
            for e in places:
                u[512 * e:512 * (e + 1)] = v.to(dt)
            w = t.full((nL,), 7.0, device="cuda")
            sem.sem_ax(h, p, u, w)
            t.cuda.synchronize()
            x = v.to(dt).double().view(1, 8, 8, 8).expand(len(places), 8, 8, 8).contiguous()
            ref = _reference(G.to(dt).double(), D, x).reshape(len(places), 512)
            for q, e in enumerate(places):
                err = (w[512 * e:512 * (e + 1)].double() - ref[q]).abs().max() / ref[q].abs().max()
                assert float(err) <= 2e-6, (p, e, float(err))
            del u, w
    finally:
        t.cuda.synchronize()
        sem.sem_destroy(h)
        t.cuda.empty_cache()
