"""Forward pass on more samples than one launch has threads for (32 threads a
sample, 2^32 threads a launch): 134 million samples of one output, 4.8 GB.
Samples are independent: the same bits as the same rows in a small batch."""
import pytest

from gpu_util import torch

pytestmark = pytest.mark.gpu


def test_forward_rows_beyond_one_launch():
    from paper_1403_0968_amd import sem
    t = torch()
    B = (1 << 27) + 37
    print(f"[gpu] network forward of {B} samples", flush=True)
    g = t.Generator(device="cuda")
    g.manual_seed(1)
    X = t.zeros(B, 16, dtype=t.bfloat16, device="cuda")
    X[:, :8] = t.randint(-8, 9, (B, 8), device="cuda", generator=g, dtype=t.int8).to(t.bfloat16)
    net = sem.sem_mlp_create(8, 128, 1, seed=3)
    try:
        Y = t.full((B + 1, 1), 7.0, device="cuda")
        sem.sem_mlp_forward(net, X, 16, B, Y)
        for r0 in (0, (1 << 26) - 20, B // 3, B - 50):
            x = X[r0:r0 + 50].contiguous()
            y = t.empty(50, 1, device="cuda")
            sem.sem_mlp_forward(net, x, 16, 50, y)
            assert t.equal(Y[r0:r0 + 50], y), r0
        assert float(Y[B]) == 7.0
    finally:
        sem.sem_mlp_destroy(net)
