"""The gradient of one training step, block by block, against FP64, with a bound
that a zero gradient and a minibatch of one sample less are shown to exceed."""
import numpy as np
import pytest
import torch

H = 256
# D, minibatch: unaligned inputs, remainders, minibatches of whole groups of 128
SIZES = [(1, 1), (1, 200), (4, 33), (30, 64), (64, 256), (100, 384), (101, 65), (256, 128), (512, 300), (520, 512)]
# of the samples' contributions: FP32 sums of at most D + 2 H + 512 terms, whose rounding is about the root of their number
# times u32, 2e-6; the rest is room for cancellation inside the network
TOL = 1e-4


def shapes(D):
    return [(H, D), (H,), (H, H), (H,), (1, H), (1,)]


def gradient(params, x, t):
    """Gradient blocks of mean (out - t)^2 in FP64, and the root of the sum of
    the samples' squared contributions to each."""
    W1, b1, W2, b2, W3, b3 = params
    gelu = torch.nn.functional.gelu
    dg = lambda a: 0.5 * (1 + torch.erf(a / np.sqrt(2))) + a * torch.exp(-a * a / 2) / np.sqrt(2 * np.pi)
    a1 = x @ W1.T + b1
    h1 = gelu(a1)
    a2 = h1 @ W2.T + b2
    h2 = gelu(a2)
    r = 2 * ((h2 @ W3.T + b3)[:, 0] - t) / x.shape[0]
    ga2 = r[:, None] * W3 * dg(a2)
    ga1 = (ga2 @ W2) * dg(a1)
    one = torch.ones_like(r)[:, None]
    parts = [(ga1, x), (ga1, one), (ga2, h1), (ga2, one), (r[:, None], h2), (r[:, None], one)]
    grads = [(a.T @ b).reshape(s) for (a, b), s in zip(parts, shapes(x.shape[1]))]
    return grads, [float(((a * a).sum(1) * (b * b).sum(1)).sum().sqrt()) for a, b in parts]


def data(D, n, seed, dev):
    g = torch.Generator(dev).manual_seed(seed)
    X = torch.randn(n, D, generator=g, dtype=torch.float64, device=dev)
    return X, -0.5 * (X * X).sum(1) + X.sin().sum(1)


@pytest.mark.parametrize("D,nb", SIZES)
def test_bound_tells_a_wrong_gradient(D, nb):
    g = torch.Generator().manual_seed(D + nb)
    he = lambda o, i: (torch.randn(o, i, generator=g, dtype=torch.float64) * np.sqrt(2.0 / i)).bfloat16().double()
    params = [he(H, D), torch.zeros(H), he(H, H), torch.zeros(H), he(1, H), torch.zeros(1)]
    params = [p.double() for p in params]
    X, lp = data(D, 700, 31 + D, "cpu")
    x, t = ((X - X.mean(0)) / X.std(0))[:nb], ((lp - lp.mean()) / lp.std())[:nb]
    grads, scale = gradient(params, x, t)
    less, _ = gradient(params, x[:-1], t[:-1]) if nb > 1 else ([0 * v for v in grads], None)
    for v, w, s in zip(grads, less, scale):
        assert float(v.norm()) > 2 * TOL * s  # a zero gradient
        assert float((v - w * (nb - 1) / nb).norm()) > 2 * TOL * s  # the last sample dropped


@pytest.mark.gpu
@pytest.mark.parametrize("D,nb", SIZES)
def test_gradient_blocks(D, nb):
    from paper_1506_05741_amd import diam

    n = 700
    X, lp = data(D, n, 31 + D, "cuda")
    s = diam.Sampler(diam.make_config(D, 4, 2, "fp32", seed=1, surrogate=1, train_max=n),
                     torch.zeros(D, dtype=torch.float64, device="cuda"), torch.eye(D, device="cuda"),
                     X[:4].contiguous())
    cut = lambda f: [v.reshape(sh) for v, sh in zip(torch.split(s.get(f).view(torch.float32).double(),
                                                               [int(np.prod(sh)) for sh in shapes(D)]), shapes(D))]
    for steps in (1, 2, 3):  # a step's minibatch is gathered by the step before
        s.surrogate_train(X, lp, steps=steps - 1, batch=nb, lr=1e-3, seed=7)
        p0, st = cut(diam.F_MLP_PARAMS), s.get(diam.F_MLP_STATS).view(torch.float32)
        s.surrogate_train(X, lp, steps=steps, batch=nb, lr=1e-3, seed=7)
        idx = s.get(diam.F_MLP_BATCH).view(torch.int32).long()[:nb]
        x = ((X[idx].float() - st[:D]) * st[D:2 * D]).double()
        t = ((lp[idx] - lp.mean()) / lp.std(correction=0)).float().double()
        grads, scale = gradient([p.bfloat16().double() for p in p0], x, t)
        for got, want, sc in zip(cut(diam.F_MLP_GRAD), grads, scale):
            assert float((got - want).norm()) <= TOL * sc, (steps, tuple(want.shape))
