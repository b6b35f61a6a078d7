"""The wave step on a grid one column wide and 270 million rows tall (4.3 GB
in place): chunks of 8 rows would need more threads than one launch holds
(2^32).  With nx = 1 the x part of the stencil is the column times the sum
of the weights; the kernel's order of operations is reproduced on windows at
both ends, in the middle and across chunk borders: equal bits."""
import numpy as np
import pytest

from gpu_util import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("r", [3, 5])
def test_tall_column(r):
    from paper_1403_0968_amd import sem
    t = torch()
    ny = 270_000_000
    print(f"[gpu] fd2d 1 x {ny} r={r}", flush=True)
    cur = t.rand(ny, 1, dtype=t.float64, device="cuda")
    nxt = t.rand(ny, 1, dtype=t.float64, device="cuda")
    w = [float(q) for q in np.asarray(sem.fd2d_weights(r))]
    dt, dx = 0.01, 0.5
    c = dt * dt / (dx * dx)
    starts = [0, 1024 - 40, ny // 2 + 3, 268_435_456 - 40, ny - 80]
    want = []
    for s in starts:
        rows = t.arange(s, s + 80, device="cuda")
        u, lap = cur[rows, 0], t.zeros(80, dtype=t.float64, device="cuda")
        for k in range(-r, r + 1):
            lap = lap + (w[r + k] * u + w[r + k] * cur[(rows + k) % ny, 0])
        want.append((2.0 * u - nxt[rows, 0]) + c * lap)
    sem.fd2d_step(cur, nxt, nxt, r, dt, dx)
    t.cuda.synchronize()
    for s, x in zip(starts, want):
        assert t.equal(nxt[s:s + 80, 0], x), s
