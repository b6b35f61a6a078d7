"""Graphs captured by a solve: one per number of iterations where a pass of its
own updates p and x (the direction has one buffer), two at an odd number in
the form of two passes (its buffers swap roles).  A child process counts the
instantiations through a library, loaded before the HIP runtime, that defines
hipGraphInstantiate and calls the runtime's."""
import os
import shutil
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

COUNTER = r"""
#include <dlfcn.h>
#include <stddef.h>
int graph_count = 0;
int hipGraphInstantiate(void **exec, void *graph, void **node, char *log, size_t n) {
  static int (*real)(void **, void *, void **, char *, size_t);
  if (!real) {
    void *h = dlopen("libamdhip64.so.7", RTLD_NOW | RTLD_NOLOAD);
    if (!h) h = dlopen("libamdhip64.so", RTLD_NOW | RTLD_NOLOAD);
    if (!h) return 999;
    real = (int (*)(void **, void *, void **, char *, size_t))dlsym(h, "hipGraphInstantiate");
  }
  graph_count += 1;
  return real(exec, graph, node, log, n);
}
"""

CHILD = r"""
import ctypes, sys
count = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
import torch as t
from paper_1403_0968_amd import sem
from seminputs import fourier_modes
out = []
for side, every in ((20, 3), (20, 4), (4, 3), (4, 4)):
    h = sem.sem_setup(7, side, side, side)
    b = t.empty(sem.sem_query(h)[1], dtype=t.float64, device="cuda")
    sem.sem_rhs(h, b, sem.SEM_SRC_FOURIER, fourier_modes(seed=1))
    x = t.zeros_like(b)
    n0 = ctypes.c_int.in_dll(count, "graph_count").value
    for _ in range(2):
        x.zero_()
        st = sem.sem_pcg_solve(h, b, x, rtol=1e-13, maxit=30, check_every=every,
                               raise_on_fail=False)
    t.cuda.synchronize()
    out.append(ctypes.c_int.in_dll(count, "graph_count").value - n0)
    sem.sem_destroy(h)
print("captures", *out, flush=True)
"""


def test_captures_per_solve(tmp_path):
    cc = shutil.which("gcc") or shutil.which("cc")
    if cc is None:
        pytest.skip("no C compiler")
    src, lib = tmp_path / "count.c", tmp_path / "libcount.so"
    src.write_text(COUNTER)
    subprocess.run([cc, "-shared", "-fPIC", str(src), "-o", str(lib), "-ldl"], check=True)
    print("[gpu] graph captures per solve", flush=True)
    r = subprocess.run([sys.executable, "-c", CHILD, str(lib)], capture_output=True, text=True,
                       timeout=100, cwd=ROOT)
    assert r.returncode == 0, r.stderr
    # streaming 20^3 (vectors of 145 MB): one; 4^3 in two passes: 2 and 1
    assert "captures 1 1 2 1" in r.stdout, r.stdout
