"""The wave step in each workgroup shape: strips of 64 x 4 (at most 0.7M
nodes), 256 x 8, 256 x 16 and 256 x 32, on either side of the lines between
them, with partial strips and chunks and grids narrower than the stencil.
The kernel multiplies and adds separately in a stated order: equal bits."""
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


@pytest.mark.parametrize("nx,ny,r", [(1, 1, 7), (5, 3, 7), (3, 70, 2), (63, 4, 1), (64, 5, 6),
                                     (65, 9, 3), (300, 7, 7), (7, 300, 4), (875, 800, 5),
                                     (875, 801, 5), (837, 839, 1), (2449, 2450, 6),
                                     (2449, 2451, 4), (2000, 3001, 2), (3465, 3463, 7),
                                     (3465, 3467, 3), (3465, 3467, 4), (3465, 3467, 7)])
def test_shapes(nx, ny, r):
    from paper_1403_0968_amd import sem
    t = torch()
    print(f"[gpu] fd2d shapes {nx}x{ny} r={r}", flush=True)
    g = t.Generator(device="cuda")
    g.manual_seed(r)
    u, v = (t.rand(ny, nx, dtype=t.float64, device="cuda", generator=g) - 0.5
            for _ in range(2))
    w = [float(q) for q in np.asarray(sem.fd2d_weights(r))]
    dt, dx = 0.01, 0.5
    c = dt * dt / (dx * dx)
    a, b = u.clone(), v.clone()
    for _ in range(2):
        a, b = _step(w, r, c, b, a), b
        a, b = b, a
    # one step into a third buffer with a value past its end
    out = t.full((nx * ny + 1,), 7.0, dtype=t.float64, device="cuda")
    sem.fd2d_step(v, u, out[:-1].view(ny, nx), r, dt, dx)
    assert t.equal(out[:-1].view(ny, nx), _step(w, r, c, v, u))
    assert float(out[-1]) == 7.0
    # two steps in place: u holds the first, v the second
    sem.fd2d_run(u, v, r, dt, dx, 2)
    assert t.equal(u, a) and t.equal(v, b)
