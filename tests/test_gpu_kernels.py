"""Kernels chosen by size, each at the sizes where it can go wrong (edges of
tiles, remainders, smallest sizes), through the public calls."""
import numpy as np
import pytest
import torch

from paper_1506_05741_amd import diam

pytestmark = pytest.mark.gpu

U64 = 2.0 ** -53


def sampler(prec, d, P, n_lag, seed, twist=None, **kw):
    """A sampler on a random Gaussian target (dense, well conditioned R) with
    its pieces: (sampler, R as the sampler holds it in FP64, mu, generator)."""
    g = torch.Generator("cuda").manual_seed(seed)
    rn = lambda *s: torch.randn(*s, generator=g, dtype=torch.float64, device="cuda")
    R, mu, x0 = torch.eye(d, dtype=torch.float64, device="cuda") + rn(d, d) / np.sqrt(d), rn(d), rn(P, d)
    if prec != "fp64":
        R = R.float()
    s = diam.Sampler(diam.make_config(d, P, n_lag, prec, seed=seed, **kw), mu, R.contiguous(), x0.contiguous(),
                     twist=twist)
    return s, R.double(), mu, rn


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("d,P", [(1, 1), (7, 16), (8, 17), (16, 2), (17, 15), (32, 33), (33, 1), (63, 16), (64, 64),
                                 (65, 3), (127, 31), (129, 65), (511, 16), (1001, 18), (1024, 130)])
def test_split_target_log_density(prec, d, P):
    """The step's target kernel for few tiles (16 x 16 per workgroup, K split)
    on accepted proposals, against FP64 products of the same operands: FP64
    within 8 d u; FP32 against the tile kernel, whose products it repeats bit
    for bit, up to the order of the FP64 row-block sum (d u, 64 blocks)."""
    twist = None
    if prec == "fp64" and d % 2 == 0:  # the twisted rows' partner lies in the same lane
        twist = torch.zeros(d, dtype=torch.float64, device="cuda")
        twist[1::2] = 0.3
    s, R, mu, rn = sampler(prec, d, P, 2, 11 + d, twist=twist, beta=0.05)
    U = torch.full((1, P), 0.5 * 2.0 ** -52, dtype=torch.float64, device="cuda")  # accepts unless log alpha < -36
    s.step_batch(1, 0.2 * rn(1, P, d), U)
    assert bool(s.get(diam.F_ACC).bool().all())
    x = s.get_f64(diam.F_X, (P, d))
    lp = s.get_f64(diam.F_LOGP, (P,))
    if prec == "fp64":
        y = (x - mu) @ R.T
        if twist is not None:
            y[:, 1::2] += twist[1::2] * y[:, 0::2] ** 2
        ref, tol = -0.5 * (y * y).sum(1), 8 * (d + 8) * U64
    else:
        t = diam.Sampler(diam.make_config(d, P, 2, prec), mu, R.float(), x.contiguous())
        ref, tol = t.get_f64(diam.F_LOGP, (P,)), 72 * U64
    assert float(((lp - ref).abs() / ref.abs()).max()) <= tol
