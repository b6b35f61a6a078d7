"""Grids whose workgroups would need 2^32 threads or more in one launch (the
rest would be dropped without an error) are refused before anything is
launched; sizes that do not fit 64 bits as a product are refused too."""
import ctypes as C
import os

import pytest

from paper_1403_0968_amd import sem


@pytest.mark.skipif(not os.path.exists(sem.LIB_PATH), reason="libsem.so not built")
@pytest.mark.parametrize("nx,ny,r", [(1, 1 << 29, 3), (1, 1 << 40, 1), (200, 1 << 29, 7),
                                     (1 << 24, 1 << 24, 2), (1 << 40, 1 << 40, 5)])
def test_refused(nx, ny, r):
    a, b = C.c_void_p(1 << 12), C.c_void_p(2 << 12)  # never read
    code = sem.lib().fd2d_step(a, b, b, nx, ny, r, 0.01, 0.5, None)
    assert code == sem.SEM_ERR_ARG
    assert b"too large" in sem.lib().sem_last_error()
