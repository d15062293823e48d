"""The whole merged second moment and mean of a window, both triangles and every
tile, against FP64 sums of the states that the window visited."""
import numpy as np
import pytest
import torch

from paper_1506_05741_amd import diam

pytestmark = pytest.mark.gpu

U64, BETA, N0 = 2.0 ** -53, 0.3, 40.0


def window(prec, d, P, n, seed):
    """(S, m) after one window, S0, x_ref and the window's stored states (K x d,
    shifted by x_ref, rounded as the window holds them)."""
    g = torch.Generator("cuda").manual_seed(seed)
    rn = lambda *s: torch.randn(*s, generator=g, dtype=torch.float64, device="cuda")
    R = torch.eye(d, dtype=torch.float64, device="cuda") + rn(d, d) / np.sqrt(d)
    s = diam.Sampler(diam.make_config(d, P, n, prec, seed=seed, beta=BETA), rn(d),
                     (R if prec == "fp64" else R.float()).contiguous(), rn(P, d).contiguous())
    A, mu = rn(d, d) / np.sqrt(d), rn(d)
    S0 = (A @ A.T + torch.eye(d, dtype=torch.float64, device="cuda") + torch.outer(mu, mu)).contiguous()
    S0 = (0.5 * (S0 + S0.T)).contiguous()
    assert s.seed_moments(S0, mu, N0)[0] == diam.OK
    x, xr = s.get_f64(diam.F_X, (P, d)).clone(), s.get_f64(diam.F_XREF, (d,)).clone()
    s.step_batch(n)
    xi = s.get(diam.F_XI).view(torch.float64 if prec == "fp64" else torch.float32)[:n * P * d].reshape(n, P, d).double()
    acc = s.get(diam.F_ACC)[:n * P].reshape(n, P, 1).bool()
    Y = torch.empty(n, P, d, dtype=torch.float64, device="cuda")
    for t in range(n):
        x = torch.where(acc[t], xr + np.sqrt(1 - BETA ** 2) * (x - xr) + xi[t], x)
        Y[t] = x - xr
    assert bool(((s.get_f64(diam.F_X, (P, d)) - x).abs() <= 8 * n * U64 * (x.abs() + xr.abs() + 1)).all())
    assert 0 < int(acc.sum()) < n * P or n * P < 64
    Y = Y.reshape(-1, d)
    Y = {"fp64": Y, "fp32": Y.float().double(), "mixed": Y.float().bfloat16().double()}[prec]
    s.merge_moments()
    return s.get_f64(diam.F_S, (d, d)).clone(), s.get_f64(diam.F_M, (d,)).clone(), S0, mu, xr, Y


def bounds(prec, S0, xr, Y, n):
    """A sum of K products in a format of unit roundoff u errs by about sqrt(K)
    u of the sum of absolute values, 8 times that allowed; the FP64 fold and the
    rebuilt states (n steps) by (8 + n) u64 of every term."""
    K, u = float(Y.shape[0]), U64 if prec == "fp64" else 2.0 ** -24
    ya = Y.abs()
    G, h, xa = ya.T @ ya, ya.sum(0), xr.abs()
    mag = G + torch.outer(h, xa) + torch.outer(xa, h) + K * torch.outer(xa, xa) + N0 * S0.abs()
    es = (8 * np.sqrt(K) * u * G + 8 * (8 + n + np.sqrt(K)) * U64 * mag) / (N0 + K)
    em = 8 * (8 + n + np.sqrt(K)) * U64 * (h + K * xa + N0 * xa) / (N0 + K)
    return es, em


def moments(S0, m0, xr, Y):
    K, h = float(Y.shape[0]), Y.sum(0)
    S = N0 * S0 + Y.T @ Y + torch.outer(h, xr) + torch.outer(xr, h) + K * torch.outer(xr, xr)
    return S / (N0 + K), (N0 * m0 + h + K * xr) / (N0 + K)


@pytest.mark.parametrize("prec,d,P,n", [("fp64", 1, 3, 9), ("fp64", 31, 40, 130), ("fp64", 64, 1024, 14),
                                        ("fp64", 65, 33, 310), ("fp64", 100, 32, 100), ("fp64", 133, 200, 41),
                                        ("fp64", 194, 256, 44), ("fp64", 451, 100, 90), ("fp64", 1030, 60, 100),
                                        ("fp64", 2050, 128, 128), ("fp64", 2051, 128, 128), ("fp32", 67, 300, 90),
                                        ("fp32", 133, 64, 66), ("fp32", 300, 100, 90), ("fp32", 602, 100, 90),
                                        ("fp32", 2052, 70, 60), ("fp32", 2051, 70, 60), ("mixed", 64, 8192, 16),
                                        ("mixed", 70, 500, 50), ("mixed", 128, 64, 130), ("mixed", 250, 100, 70),
                                        ("mixed", 512, 256, 40)])
def test_whole_moments_of_a_window(prec, d, P, n):
    S, m, S0, m0, xr, Y = window(prec, d, P, n, 5 + d)
    es, em = bounds(prec, S0, xr, Y, n)
    Sr, mr = moments(S0, m0, xr, Y)
    assert bool(((S - Sr).abs() <= es).all()) and bool(((m - mr).abs() <= em).all())
    # the bound tells: one sample left out exceeds it, of more than 100000 the smallest split
    out = 1 if Y.shape[0] < 100000 else Y.shape[0] // 64
    less, _ = moments(S0, m0, xr, torch.cat([Y[:-out], 0 * Y[-out:]]))
    assert bool(((less - Sr).abs() > es).any())
