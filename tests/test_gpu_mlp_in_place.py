"""Outputs that lie over the network's input: the forward pass and the gradient
read every sample before they write (the outputs were the last thing written
by the calls that had a launch per product)."""
import pytest

from gpu_util import torch

pytestmark = pytest.mark.gpu


def _input(B, ld, seed):
    t = torch()
    g = t.Generator(device="cuda")
    g.manual_seed(seed)
    X = t.randn(B, ld, device="cuda", generator=g)
    X[:, 8:] = 0
    return X.to(t.bfloat16)


@pytest.mark.parametrize("fp32", [0, 1])
@pytest.mark.parametrize("K,shift", [(8, 0), (27, 0), (1, 32), (8, 16)])
def test_forward_over_its_input(K, shift, fp32):
    from paper_1403_0968_amd import sem
    t = torch()
    B, n = 20000, K * (K + 1) // 2
    print(f"[gpu] forward in place K={K} shift={shift} fp32={fp32}", flush=True)
    net = sem.sem_mlp_create(8, 128, n, seed=5)
    sem.sem_mlp_set_precision(net, sem.SEM_FP32 if fp32 else sem.SEM_BF16)
    try:
        X = _input(B, 16, 1)
        Y = t.empty(B, n, device="cuda")
        sem.sem_mlp_forward(net, X, 16, B, Y)
        # X at `shift` bytes into a buffer that Y fills from its start
        buf = t.zeros(max(B * n, B * 8) + 64, device="cuda")
        x = buf.view(t.bfloat16)[shift // 2:][:B * 16].view(B, 16)
        y = buf[:B * n].view(B, n)
        for _ in range(3):
            x.copy_(X)
            sem.sem_mlp_forward(net, x, 16, B, y)
            assert t.equal(y, Y)
    finally:
        sem.sem_mlp_destroy(net)


@pytest.mark.parametrize("fp32", [0, 1])
def test_gradient_over_its_input(fp32):
    from paper_1403_0968_amd import sem
    t = torch()
    K, B = 8, 4096
    print(f"[gpu] gradient in place fp32={fp32}", flush=True)
    net = sem.sem_mlp_create(8, 128, 36, seed=5)
    sem.sem_mlp_set_precision(net, sem.SEM_FP32 if fp32 else sem.SEM_BF16)
    try:
        npar = sem.sem_mlp_info(net)["n_params"]
        X = _input(B, 16, 2)
        T = t.rand(B, 2 * K, device="cuda")
        G = t.empty(npar, device="cuda")
        loss = sem.sem_mlp_loss_grad_factor(net, X, 16, T, K, B, G)
        buf = t.zeros(max(npar, B * 8), device="cuda")
        x = buf.view(t.bfloat16)[:B * 16].view(B, 16)
        x.copy_(X)
        assert sem.sem_mlp_loss_grad_factor(net, x, 16, T, K, B, buf[:npar]) == loss
        t.cuda.synchronize()
        assert t.equal(buf[:npar], G)
    finally:
        sem.sem_mlp_destroy(net)
