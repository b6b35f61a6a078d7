"""The wave step's workgroup shape by the sides of the grid: on either side of
each line (64 columns, strips a multiple of 8, rows 32, 64 and 512, threads
and nodes), with partial strips and chunks.  The kernel multiplies and adds
separately in a stated order: equal bits."""
import numpy as np
import pytest

from gpu_util import torch

pytestmark = pytest.mark.gpu


def _step(w, r, c, cur, prev):
    t = torch()
    lap = t.zeros_like(cur)
    for k in range(-r, r + 1):
        lap = lap + (w[r + k] * t.roll(cur, -k, 1) + w[r + k] * t.roll(cur, -k, 0))
    return (2.0 * cur - prev) + c * lap


@pytest.mark.parametrize("nx,ny,r", [(1, 2000003, 3), (64, 30001, 7), (65, 30001, 7),
                                     (2047, 1501, 4), (2048, 1501, 4), (2048, 1501, 5),
                                     (2049, 1501, 4), (4001, 511, 2), (4001, 512, 2),
                                     (1536, 1627, 2), (1536, 1628, 2), (1536, 1953, 3),
                                     (1536, 1954, 3), (47000, 32, 5), (50000, 31, 5),
                                     (24001, 63, 6), (24001, 64, 6), (1000, 5070, 7),
                                     (1000, 5090, 7), (1023, 5500, 3), (1024, 5500, 3),
                                     (131000, 16, 7), (3000001, 5, 1),
                                     (7001, 7201, 2), (7001, 7201, 4), (7001, 7101, 4),
                                     (8192, 6105, 4), (8192, 6103, 4), (8192, 6105, 3)])
def test_sides(nx, ny, r):
    from paper_1403_0968_amd import sem
    t = torch()
    print(f"[gpu] fd2d sides {nx}x{ny} r={r}", flush=True)
    g = t.Generator(device="cuda")
    g.manual_seed(r)
    u, v = (t.rand(ny, nx, dtype=t.float64, device="cuda", generator=g) - 0.5
            for _ in range(2))
    w = [float(q) for q in np.asarray(sem.fd2d_weights(r))]
    dt, dx = 0.01, 0.5
    c = dt * dt / (dx * dx)
    out = t.full((nx * ny + 1,), 7.0, dtype=t.float64, device="cuda")
    sem.fd2d_step(v, u, out[:-1].view(ny, nx), r, dt, dx)
    assert t.equal(out[:-1].view(ny, nx), _step(w, r, c, v, u))
    assert float(out[-1]) == 7.0
