"""The DG volume term with one wave per workgroup (blocked layout, and
element-major up to 32768 triangles) and with four: element counts around
whole blocks of 16, whole workgroups and the line."""
import pytest

from test_gpu_dg import _check_volume, _setup

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,nx,ny", [(1, 1, 1), (4, 4, 2), (8, 3, 3), (3, 4, 8), (6, 11, 3),
                                     (2, 128, 128), (2, 129, 127), (2, 127, 130), (5, 2, 8193)])
def test_volume(N, nx, ny):
    """Error bound of the volume term's other tests; both layouts the same bits."""
    from paper_1403_0968_amd import sem
    print(f"[gpu] dg waves N={N} {2 * nx * ny} triangles", flush=True)
    h, ops, geo, X, Y, B, Q = _setup(sem, N, nx, ny)
    try:
        assert _check_volume(sem, h, ops, geo, B, Q)[0] <= 1e-13
    finally:
        sem.dg_destroy(h)
