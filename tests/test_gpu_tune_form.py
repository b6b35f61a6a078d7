"""The tuner times the operator in the form that the batch's iterations run:
the profiler's kernel names carry the form (k_bax's fifth template argument:
2 the direction and its sums inside, 3 a pass of its own for p and x).  The
tuned batch gives the bits of the single solves, and a cache entry of a file
without forms is kept and not read."""
import json
import os
import re

import pytest

from seminputs import fourier_modes

from gpu_util import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("side,want", [(3, 2), (19, 3)])
def test_tuned_form_is_the_iterations(side, want, tmp_path):
    from paper_1403_0968_amd import sem
    t = torch()
    print(f"[gpu] tuned form side={side}", flush=True)
    hs = [sem.sem_setup(7, side, side, side, mapping=sem.SEM_MAP_SINE_CYCLIC),
          sem.sem_setup(7, side, side, 2)]
    bt = sem.sem_batch_create(hs)
    path = str(tmp_path / "tune.json")
    os.environ["SEM_AUTOTUNE_CACHE"] = path
    try:
        bs = []
        for h in hs:
            b = t.empty(sem.sem_query(h)[1], dtype=t.float64, device="cuda")
            sem.sem_rhs(h, b, sem.SEM_SRC_FOURIER, fourier_modes(seed=2))
            bs.append(b)
        with t.profiler.profile(activities=[t.profiler.ProfilerActivity.CPU,
                                            t.profiler.ProfilerActivity.CUDA]) as prof:
            b1, g1, us = sem.sem_batch_tune(bt, sem.SEM_FP64)
            t.cuda.synchronize()
        assert us > 0
        forms = set()
        for e in prof.events():
            m = re.search(r"k_bax<\d+, double, double, double, (\d)", e.name)
            if m:
                forms.add(int(m.group(1)))
        assert forms == {want}, forms
        # an entry as older files name it, and the one just written
        cache = json.load(open(path))
        (key, val), = cache.items()
        old = key[:key.index("|form")]
        other = [64 if val[0] != 64 else 128, 4]
        json.dump({old: other}, open(path, "w"), indent=1)
        txt = open(path).read()
        open(path, "w").write(re.sub(r"\[\s*(\d+),\s*(\d+)\s*\]", r"[\1, \2]", txt))
        assert sem.sem_batch_tune(bt, sem.SEM_FP64)[2] > 0
        cache = json.load(open(path))
        assert cache[old] == other and key in cache
        assert sem.sem_batch_tune(bt, sem.SEM_FP64)[2] == -1.0
        kw = dict(rtol=1e-9, maxit=9, check_every=4, raise_on_fail=False)
        xs = [t.zeros_like(b) for b in bs]
        sem.sem_batch_pcg_solve(bt, bs, xs, **kw)
        for h, b, x in zip(hs, bs, xs):
            y = t.zeros_like(b)
            sem.sem_pcg_solve(h, b, y, **kw)
            t.cuda.synchronize()
            assert bool(y.abs().max() > 0) and t.equal(x, y)
    finally:
        del os.environ["SEM_AUTOTUNE_CACHE"]
        sem.sem_batch_destroy(bt)
        for h in hs:
            sem.sem_destroy(h)
