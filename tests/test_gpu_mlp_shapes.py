"""The correction network's kernels at the edges of their tiles (16 samples,
16 outputs, 32 inputs, waves dealt four samples at a time), against the FP64
oracle.

Tolerances.  FP32: the products of a layer are sums of at most 512 FP32
terms, each sum off by about sqrt(512) 2^-24 = 1.4e-6 of the terms' norm,
through three layers forward and three back: 2e-5 of the block's largest
entry.  BF16: hidden activations rounded to 2^-9 at two layers, averaged over
128 inputs: 2e-2 of the largest entry."""
import numpy as np
import pytest

from oracle import mlp
from seminputs import normal

from gpu_util import bf16_round, to_dev, to_host, torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sem():
    from paper_1403_0968_amd import sem as s
    s.lib()
    return s


def _net(sem, n_in, n_out, prec, seed):
    net = sem.sem_mlp_create(n_in, 128, n_out, seed=seed)
    if prec == "fp32":
        sem.sem_mlp_set_precision(net, sem.SEM_FP32)
    params = sem.sem_mlp_get_params(net)
    W1, b1, W2, b2, W3, b3 = mlp.unpack(params.astype(np.float64), n_in, 128, n_out)
    at = 0
    for blk, amount in ((W1, 0), (b1, .1), (W2, 0), (b2, .1), (W3, 0), (b3, .1)):
        n = np.asarray(blk).size
        if amount:
            params[at:at + n] = normal(n, seed=seed + at) * amount
        at += n
    sem.sem_mlp_set_params(net, params)
    th = params.astype(np.float64)
    if prec == "bf16":  # the weights the forward and backward products use
        at = 0
        for blk in (W1, b1, W2, b2, W3, b3):
            n = np.asarray(blk).size
            if np.asarray(blk).ndim == 2:
                th[at:at + n] = bf16_round(th[at:at + n])[0]
            at += n
    return net, th


def _inputs(B, n_in, ldx, seed):
    x = np.zeros((B, ldx))
    x[:, :n_in] = normal((B, n_in), seed=seed)
    return bf16_round(x)


@pytest.mark.parametrize("prec", ["bf16", "fp32"])
@pytest.mark.parametrize("B,n_in,n_out", [(1, 8, 378), (16, 8, 16), (17, 1, 17), (15, 33, 1),
                                          (33, 16, 129), (50, 100, 1024)])
def test_forward(sem, B, n_in, n_out, prec):
    print(f"[gpu] mlp forward B={B} n_in={n_in} n_out={n_out} {prec}", flush=True)
    t = torch()
    net, th = _net(sem, n_in, n_out, prec, seed=B)
    try:
        ldx = sem.sem_mlp_info(net)["n_in_padded"] + 16  # a row stride beyond the padding
        xb, u16 = _inputs(B, n_in, ldx, seed=B + 1)
        Y = t.full((B + 1, n_out), 7.0, dtype=t.float32, device="cuda")
        sem.sem_mlp_forward(net, to_dev(u16.view(np.int16), t.int16), ldx, B, Y)
        t.cuda.synchronize()
        got = to_host(Y).astype(np.float64)
        assert (got[B] == 7.0).all()  # nothing past the last sample
        ref = mlp.forward(th, xb[:, :n_in], n_in, 128, n_out)
        rel = np.max(np.abs(got[:B] - ref)) / np.max(np.abs(ref))
        print(f"[mlp fwd] {rel:.2e}")
        assert rel <= (2e-5 if prec == "fp32" else 2e-2)
    finally:
        sem.sem_mlp_destroy(net)


@pytest.mark.parametrize("K", [1, 8, 27])
@pytest.mark.parametrize("B", [1, 4, 31, 33, 300])
def test_factor_gradient_fp32(sem, K, B):
    print(f"[gpu] factor gradient K={K} B={B}", flush=True)
    t = torch()
    no = K * (K + 1) // 2
    net, th = _net(sem, 8, no, "fp32", seed=5 + K)
    try:
        # a pre-activation within rounding of 0 has no defined relu mask: the
        # first seed whose pre-activations all stay clear of it
        W1, b1, W2, b2 = mlp.unpack(th, 8, 128, no)[:4]
        for seed in range(B, B + 50):
            xb, u16 = _inputs(B, 8, 16, seed=seed)
            z1 = xb[:, :8] @ W1.T + b1
            z2 = np.maximum(z1, 0) @ W2.T + b2
            if min(np.abs(z1).min(), np.abs(z2).min()) > 5e-6:
                break
        T = np.concatenate([normal((B, K), seed=31), normal((B, K), seed=32) * 0.1],
                           1).astype(np.float32)
        g = t.empty(th.size, dtype=t.float32, device="cuda")
        loss = sem.sem_mlp_loss_grad_factor(net, to_dev(u16.view(np.int16), t.int16), 16,
                                            to_dev(T, t.float32), K, B, grad=g)
        t.cuda.synchronize()
        lo, go = mlp.factor_net_loss_and_grad(th, xb[:, :8], T[:, :K].astype(np.float64),
                                              T[:, K:].astype(np.float64), 8, 128, K)
        assert abs(loss - lo) <= 2e-5 * lo
        gg = to_host(g).astype(np.float64)
        for name, a, b in zip(("W1", "b1", "W2", "b2", "W3", "b3"),
                              mlp.unpack(gg, 8, 128, no), mlp.unpack(go, 8, 128, no)):
            worst = np.max(np.abs(a - b)) / np.max(np.abs(b))
            print(f"[factor grad] {name} {worst:.1e}")
            assert worst <= 2e-5, name
        # without a buffer the network keeps the gradient for Adam
        p0 = sem.sem_mlp_get_params(net)
        sem.sem_mlp_loss_grad_factor(net, to_dev(u16.view(np.int16), t.int16), 16,
                                     to_dev(T, t.float32), K, B)
        sem.sem_mlp_adam(net, None, lr=1e-3)
        t.cuda.synchronize()
        new = sem.sem_mlp_get_params(net).astype(np.float64)
        ref, _, _ = mlp.adam_step(p0.astype(np.float64), gg, np.zeros_like(gg),
                                  np.zeros_like(gg), 1, 1e-3)
        assert np.max(np.abs(new - ref)) <= 1e-6 * np.max(np.abs(ref))
    finally:
        sem.sem_mlp_destroy(net)
