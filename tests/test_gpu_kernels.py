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
                                 (65, 3), (127, 31), (129, 65), (511, 16), (1001, 18), (1024, 130),
                                 (1026, 290), (4100, 70), (1030, 960), (1031, 770)])
def test_target_log_density_by_size(prec, d, P):
    """The step's target kernels (16 x 16 per workgroup with K split, 32- and
    64-row tiles of the direct-to-LDS engine, the tile kernel) on accepted
    proposals, against FP64 products of the same operands: FP64 within 8 d u;
    FP32 against the tile kernel at initialisation, whose products they repeat
    bit for bit, up to the order of the FP64 row-block sum (d u, 64 blocks)."""
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


@pytest.mark.parametrize("d,P,n,nproj,proposal", [(1, 1, 3, 1, "diam"), (2, 5, 65, 4, "diam"), (31, 3, 130, 0, "am"),
                                                  (32, 16, 64, 2, "diam"), (63, 2, 33, 4, "diam"),
                                                  (64, 4, 66, 4, "diam"), (65, 3, 1, 1, "diam"),
                                                  (100, 20, 70, 4, "diam"), (128, 5, 34, 3, "pcn"),
                                                  (129, 2, 35, 4, "diam"), (191, 3, 7, 1, "am"),
                                                  (192, 300, 36, 4, "diam"), (193, 3, 9, 2, "diam"),
                                                  (130, 1025, 3, 1, "diam"), (66, 8193, 2, 1, "diam")])
def test_steps_of_a_call_in_one_launch(d, P, n, nproj, proposal):
    """The loop with R in registers and the launches per step past its range: states, log densities, log ratios, traced projections and decisions of
    two calls against the recursion in FP64 on the directions the call drew.
    The recursion contracts (rho <= 1), so t steps err by at most t times one
    step's 4 u, and log pi by 8 (d + n) u of the sum of its absolute terms."""
    twist = None
    if d % 2 == 0:
        twist = torch.zeros(d, dtype=torch.float64, device="cuda")
        twist[1::2] = 0.2
    s, R, mu, rn = sampler("fp64", d, P, n + 2, 77 + d, twist=twist, beta=0.25, proposal=proposal)
    walk = proposal == "am"
    rho, c = (1.0 if walk else np.sqrt(1 - 0.25 ** 2)), 0.25
    proj = rn(nproj, d) if nproj else None
    trace = torch.zeros(n + 2, 1 + nproj, P, dtype=torch.float64, device="cuda")
    s.set_trace(proj, trace)
    scale = 0.4 / np.sqrt(d)
    done, tot = 0, 0.0
    for m in (2, n):
        x, z = s.get_f64(diam.F_X, (P, d)), s.get_f64(diam.F_Z, (P, d))
        lp, xr = s.get_f64(diam.F_LOGP, (P,)), s.get_f64(diam.F_XREF, (d,))
        W = (scale * rn(m, P, d)).contiguous()
        U = torch.rand(m, P, dtype=torch.float64, device="cuda").clamp_(1e-12)
        cnt = torch.full((P,), 7, dtype=torch.int32, device="cuda")
        s.step_batch(m, W, U, cnt)
        Xi = s.get(diam.F_XI).view(torch.float64)[:m * P * d].reshape(m, P, d)
        La = s.get(diam.F_LA).view(torch.float64)[:m * P].reshape(m, P)
        Acc = s.get(diam.F_ACC)[:m * P].reshape(m, P).bool()
        assert torch.equal(cnt, 7 + Acc.sum(0, dtype=torch.int32))
        mag = torch.maximum(x.abs(), z.abs()).amax() + Xi.abs().amax() * m + mu.abs().amax()
        for t in range(m):
            xp, zp = xr + rho * (x - xr) + Xi[t], rho * z + c * W[t]
            y = (xp - mu) @ R.T
            ya = (xp - mu).abs() @ R.abs().T
            if twist is not None:
                ya[:, 1::2] += 3 * twist[1::2] * ya[:, 0::2] ** 2
                y[:, 1::2] += twist[1::2] * y[:, 0::2] ** 2
            lpp = -0.5 * (y * y).sum(1)
            tol = 8 * (d + m + 8) * U64 * ((y.abs() * ya).sum(1) + (y.abs() + ya) @ R.abs().sum(1) * mag)
            q = 0.0 if walk else 0.5 * ((zp * zp).sum(1) - (z * z).sum(1))
            la = lpp - lp + q
            assert bool(((La[t] - la).abs() <= 2 * tol + 8 * (d + m) * U64 * (1 + (zp * zp).sum(1))).all())
            assert torch.equal(Acc[t], torch.log(U[t]) < La[t])
            a = Acc[t][:, None]
            x, z, lp = torch.where(a, xp, x), torch.where(a, zp, z), torch.where(Acc[t], lpp, lp)
            tot = tot + x.sum(0)
            assert bool(((trace[done + t, 0] - lp).abs() <= 2 * tol + 8 * (d + m) * U64 * lp.abs()).all())
            for k in range(nproj):
                bound = 4 * (d + m) * U64 * proj[k].abs().sum() * mag
                assert bool(((trace[done + t, 1 + k] - x @ proj[k]).abs() <= bound).all())
        assert 0 < int(Acc.sum()) or m * P < 8
        assert bool(((s.get_f64(diam.F_X, (P, d)) - x).abs() <= 4 * m * U64 * mag).all())
        assert bool(((s.get_f64(diam.F_Z, (P, d)) - z).abs() <= 4 * m * U64 * mag).all())
        assert bool(((s.get_f64(diam.F_LOGP, (P,)) - lp).abs() <= 2 * tol + 8 * (d + m) * U64 * lp.abs()).all())
        done += m
    s.merge_moments()  # the window store of both calls
    K = (n + 2) * P
    assert bool(((s.get_f64(diam.F_M, (d,)) - tot / K).abs() <= 4 * (K + n) * U64 * mag).all())


@pytest.mark.parametrize("prec,d,P,n", [("fp64", 2, 3, 2), ("fp64", 30, 33, 3), ("fp64", 32, 8, 40), ("fp64", 62, 5, 7),
                                        ("fp64", 66, 17, 31), ("fp64", 130, 64, 33), ("fp64", 75, 9, 5),
                                        ("fp64", 194, 256, 44), ("fp64", 2050, 128, 128), ("fp32", 4, 3, 2),
                                        ("fp32", 28, 65, 3), ("fp32", 68, 31, 9), ("fp32", 132, 64, 66),
                                        ("fp32", 300, 100, 90), ("fp32", 70, 9, 5),
                                        ("fp64", 1, 3, 9), ("fp64", 3, 2, 3), ("fp64", 65, 17, 31),
                                        ("fp64", 129, 64, 33), ("fp64", 451, 100, 90), ("fp64", 2051, 128, 128),
                                        ("fp32", 1, 3, 9), ("fp32", 67, 31, 9), ("fp32", 133, 64, 66),
                                        ("fp32", 602, 100, 90)])
def test_proposal_and_scatter_products(prec, d, P, n):
    """The proposal contraction and the merged moments at the edges of their
    tiles and sizes of the dispatch, against FP64 products of the same operands
    (factor, normals, visited states as the sampler holds them).  A sum of k
    terms in a format of unit roundoff u errs by at most k u sum |a b|; the
    window store rounds each entry once more in FP32."""
    s, R, mu, rn = sampler(prec, d, P, n, 5 + d, beta=0.3)
    A = rn(d, d) / np.sqrt(d)
    S0 = A @ A.T + torch.eye(d, dtype=torch.float64, device="cuda") + torch.outer(mu, mu)
    N0 = 50.0
    assert s.seed_moments(S0.contiguous(), mu, N0)[0] == diam.OK
    L, xr = s.get_f64(diam.F_L, (d, d)).T, s.get_f64(diam.F_XREF, (d,))
    wt, u = (torch.float64, U64) if prec == "fp64" else (torch.float32, 2.0 ** -24)
    X = torch.empty(n, P, d, dtype=torch.float64, device="cuda")
    if n > 8:  # all steps in one call: the contraction's columns
        s.step_batch(n)
        W = s.get(diam.F_W).view(wt).reshape(n * P, d).double()
        Xi = s.get(diam.F_XI).view(wt).reshape(n * P, d).double()
        ref, mag = 0.3 * (W @ L.T), 0.3 * (W.abs() @ L.abs().T)
        assert bool(((Xi - ref).abs() <= (d + 4) * u * mag + 1e-300).all())
        s.merge_moments()
        S = s.get_f64(diam.F_S, (d, d))
        assert torch.equal(S, S.T) and bool(torch.isfinite(S).all())
        return
    for t in range(n):
        s.step_batch(1, rn(1, P, d))
        X[t] = s.get_f64(diam.F_X, (P, d))
    s.merge_moments()
    Y, K = X.reshape(-1, d) - xr, float(n * P)
    scale = 2 * (K + 8) * u * (Y.abs().T @ Y.abs() + 2 * torch.outer(Y.abs().sum(0), xr.abs()) +
                               K * torch.outer(xr.abs(), xr.abs())) + 8 * U64 * N0 * S0.abs()
    ref = (N0 * S0 + X.reshape(-1, d).T @ X.reshape(-1, d)) / (N0 + K)
    assert bool(((s.get_f64(diam.F_S, (d, d)) - ref).abs() * (N0 + K) <= scale + scale.T).all())


@pytest.mark.parametrize("prec,d,P,n", [("fp64", 1, 1, 2), ("fp64", 63, 3, 2), ("fp64", 66, 130, 65),
                                        ("fp64", 129, 2, 4100), ("fp32", 200, 100, 90), ("mixed", 128, 64, 130)])
def test_merge_by_size(prec, d, P, n):
    """S and m after a merge from the kernel's own splits, tiles and both
    triangles, against FP64 sums over the visited states: (K + 8) u of the sums
    of absolute values in the window's format, the mean's likewise."""
    s, R, mu, rn = sampler(prec, d, P, n, 17 + d, beta=0.3)
    S0 = torch.eye(d, dtype=torch.float64, device="cuda") + torch.outer(mu, mu)
    assert s.seed_moments(S0.contiguous(), mu, 40.0)[0] == diam.OK
    proj = torch.eye(d, dtype=torch.float64, device="cuda")[:, :min(d, 4)].T.contiguous()
    trace = torch.zeros(n, 1 + proj.shape[0], P, dtype=torch.float64, device="cuda")
    s.set_trace(proj, trace)
    m0 = s.get_f64(diam.F_M, (d,)).clone()
    s.step_batch(n)
    s.merge_moments()
    S, m, K = s.get_f64(diam.F_S, (d, d)), s.get_f64(diam.F_M, (d,)), float(n * P)
    x = trace[:, 1:].permute(1, 0, 2).reshape(proj.shape[0], -1)
    q, u = proj.shape[0], {"fp64": U64, "fp32": 2.0 ** -24, "mixed": 2.0 ** -8}[prec]
    assert torch.equal(S, S.T)
    y = x - m0[:q, None]
    err = 2 * (K + 8) * U64 * (x.abs().sum(1) + 40 * m0[:q].abs()) + 2 * u * y.abs().sum(1)
    assert bool((((40.0 * m0[:q] + x.sum(1)) / (40.0 + K) - m[:q]).abs() * (40.0 + K) <= err).all())
    ref = (40.0 * S0[:q, :q] + x @ x.T) / (40.0 + K)
    mag = x.abs() @ x.abs().T + 40 * S0[:q, :q].abs() + K * torch.outer(m0[:q].abs(), m0[:q].abs())
    acc = U64 if prec == "fp64" else 2.0 ** -24
    err = 4 * (min(K, 4096) + 8) * acc * mag + 4 * u * (y.abs() @ y.abs().T + y.abs().sum(1)[:, None] * m0[:q].abs() +
                                                       (y.abs().sum(1)[:, None] * m0[:q].abs()).T)
    assert bool(((ref - S[:q, :q]).abs() * (40.0 + K) <= err).all())


@pytest.mark.parametrize("prec,d", [("fp64", 1), ("fp64", 15), ("fp64", 17), ("fp64", 48), ("fp64", 63), ("fp64", 64),
                                    ("fp64", 66), ("fp64", 127), ("fp64", 129), ("fp64", 320), ("fp64", 451),
                                    ("fp32", 200), ("fp64", 1030)])
def test_refactorisation_by_size(prec, d):
    """L L^T against the covariance it factors, entry by entry: (d + 8) u of
    |L| |L^T| (block inverses: times their condition, here below 8), and once
    more the FP32 rounding of L where it is rounded."""
    s, R, mu, rn = sampler(prec, d, 3, 2, 13 + d, beta=0.3)
    A = 0.3 * rn(d, d) / np.sqrt(d)
    C = A @ A.T + torch.eye(d, dtype=torch.float64, device="cuda")
    S0 = C + torch.outer(mu, mu)
    assert s.seed_moments(S0.contiguous(), mu, 50.0)[0] == diam.OK
    L = s.get_f64(diam.F_L, (d, d)).T
    assert torch.equal(L, torch.tril(L))
    u = 8 * (d + 8) * U64 + (0 if prec == "fp64" else 4 * 2.0 ** -24)
    assert bool(((L @ L.T - (S0 - torch.outer(mu, mu))).abs() <= u * (L.abs() @ L.abs().T) + 8 * U64 * S0.abs()).all())


@pytest.mark.parametrize("prec,d,P", [("fp64", 1, 1), ("fp64", 15, 17), ("fp64", 64, 16), ("fp64", 65, 15),
                                      ("fp64", 130, 33), ("fp32", 511, 20), ("fp64", 512, 64), ("fp64", 577, 3),
                                      ("fp64", 1023, 18), ("fp64", 1024, 31), ("fp64", 1025, 17), ("fp32", 2051, 5)])
def test_whitening_by_size(prec, d, P):
    """Z = L^-1 (x - x_ref) and its column norms after a refactorisation, all
    rows in one launch up to d = 1024 and in pieces above: the solve's backward
    error is bounded by d u |L| |Z| per entry (block inverses: times the
    blocks' condition, here below 8)."""
    s, R, mu, rn = sampler(prec, d, P, 2, 3 + d, beta=0.3)
    A = 0.3 * rn(d, d) / np.sqrt(d)
    S0 = A @ A.T + torch.eye(d, dtype=torch.float64, device="cuda") + torch.outer(mu, mu)
    assert s.seed_moments(S0.contiguous(), mu, 50.0)[0] == diam.OK
    L, xr = s.get_f64(diam.F_L, (d, d)).T, s.get_f64(diam.F_XREF, (d,))
    X, Z, zq = s.get_f64(diam.F_X, (P, d)), s.get_f64(diam.F_Z, (P, d)), s.get_f64(diam.F_ZQ, (P,))
    assert bool(((Z @ L.T - (X - xr)).abs() <= 8 * (d + 8) * U64 * (Z.abs() @ L.abs().T + X.abs() + xr.abs())).all())
    assert bool(((zq - (Z * Z).sum(1)).abs() <= (d + 8) * U64 * zq).all())


@pytest.mark.parametrize("d,P,M", [(65, 3, 2), (130, 17, 2), (1100, 4, 2)])
def test_per_chain_whitening(d, P, M):
    """Every chain's Z after a local update against its own pair, as above."""
    s, R, mu, rn = sampler("fp64", d, P, 4, 9 + d, beta=0.3, M=M)
    S0 = torch.eye(d, dtype=torch.float64, device="cuda") + torch.outer(mu, mu)
    assert s.seed_moments(S0.contiguous(), mu, 50.0)[0] == diam.OK
    s.step_batch(4)
    s.merge_moments()
    assert s.update_proposal()[0] == diam.OK
    Lp, xrp = s.get_f64(diam.F_LP, (P, d, d)), s.get_f64(diam.F_XREFP, (P, d))
    X, Z = s.get_f64(diam.F_X, (P, d)), s.get_f64(diam.F_Z, (P, d))
    for p in range(P):
        L = torch.tril(Lp[p].T)
        y, m = L @ Z[p] - (X[p] - xrp[p]), L.abs() @ Z[p].abs() + X[p].abs() + xrp[p].abs()
        assert bool((y.abs() <= 8 * (d + 8) * U64 * m).all())


@pytest.mark.parametrize("D,nb", [(1, 1), (4, 33), (30, 64), (64, 256), (101, 65), (512, 300), (520, 512)])
def test_training_step_by_size(D, nb):
    """Gradient and Adam step of one minibatch at the sizes of the network's
    product kernels (unaligned inputs on the element engine), against FP64
    products of the same rounded weights.  A gradient entry is a chain of at
    most three products of D, 256 and nb terms in FP32: (D + 512 + nb) u of the
    gradient with every factor taken positive, doubled for the activations'
    own rounding; Adam's first step is lr g / (|g| + eps) up to 8 u."""
    H, n = 256, 700
    s, R, mu, rn = sampler("fp32", D, 4, 2, 31 + D, surrogate=1, train_max=n)
    X = rn(n, D)
    lp = -0.5 * (X * X).sum(1) + X.sin().sum(1)
    shapes = [(H, D), (H,), (H, H), (H,), (1, H), (1,)]
    cut = lambda f: [t.reshape(sh) for t, sh in zip(torch.split(s.get(f).view(torch.float32).double(),
                                                                [int(np.prod(sh)) for sh in shapes]), shapes)]
    dg = lambda a: 0.5 * (1 + torch.erf(a / np.sqrt(2))) + a * torch.exp(-a * a / 2) / np.sqrt(2 * np.pi)
    for steps in (1, 2):  # the second step's minibatch is gathered by the first
        s.surrogate_train(X, lp, steps=steps - 1, batch=nb, lr=1e-3, seed=7)
        p0, st = cut(diam.F_MLP_PARAMS), s.get(diam.F_MLP_STATS).view(torch.float32)
        s.surrogate_train(X, lp, steps=steps, batch=nb, lr=1e-3, seed=7)
        g, p1, idx = cut(diam.F_MLP_GRAD), cut(diam.F_MLP_PARAMS), s.get(diam.F_MLP_BATCH).view(torch.int32).long()
        W1, b1, W2, b2, W3, b3 = [p.bfloat16().double() for p in p0]
        x = ((X[idx].float() - st[:D]) * st[D:2 * D]).double()
        t = ((lp[idx] - lp.mean()) / lp.std(correction=0)).float().double()
        a1 = x @ W1.T + b1
        h1 = torch.nn.functional.gelu(a1)
        a2 = h1 @ W2.T + b2
        h2 = torch.nn.functional.gelu(a2)
        r = 2 * ((h2 @ W3.T + b3)[:, 0] - t) / nb
        ga2 = r[:, None] * W3 * dg(a2)
        ga1 = (ga2 @ W2) * dg(a1)
        ref = [ga1.T @ x, ga1.sum(0), ga2.T @ h1, ga2.sum(0), (r @ h2)[None], r.sum()[None]]
        # every factor positive, residuals with the size of their terms
        ra = (2 * (h2.abs() @ W3.abs().T + b3.abs())[:, 0] + 2 * t.abs()) / nb
        m2 = ra[:, None] * W3.abs() * 1.2
        m1 = (m2 @ W2.abs()) * 1.2
        xa, ha1 = x.abs() + 1e-3, x.abs() @ W1.abs().T + b1.abs() + 1e-3
        ha2 = ha1 @ W2.abs().T + b2.abs()
        mag = [m1.T @ xa, m1.sum(0), m2.T @ ha1, m2.sum(0), (ra @ ha2)[None], ra.sum()[None]]
        # the activations' rounding, relative to their own terms, moves gelu and gelu'
        amp = 1 + float(ha2.max())
        for got, want, m, q0, q1 in zip(g, ref, mag, p0, p1):
            assert bool(((got - want).abs() <= 2 * (D + 512 + nb) * 2.0 ** -24 * amp * m).all())
            if steps == 1:
                step = 1e-3 * got / (got.abs() + 1e-8)
                assert bool(((q0 - q1 - step).abs() <= 1e-3 * 32 * 2.0 ** -24 + 2.0 ** -24 * q0.abs()).all())


@pytest.mark.parametrize("n_obs,d,P", [(1, 4, 1), (63, 8, 3), (65, 36, 65), (200, 12, 64), (131, 33, 17),
                                       (131072, 32, 66), (131200, 40, 3)])
def test_logistic_target_by_size(n_obs, d, P):
    """The logistic target's tiles (64 and 128 observations, the unaligned
    fallback) against FP64 at the accepted states: an FP32 dot product of d
    terms errs by d u32 sum |a x|, a term of the log likelihood by no more than
    that plus 4 u32 (|t| + 1) of its own evaluation."""
    g = torch.Generator("cuda").manual_seed(n_obs + d)
    rn = lambda *s: torch.randn(*s, generator=g, dtype=torch.float64, device="cuda")
    A, y = (rn(n_obs, d) / np.sqrt(d)).float(), (rn(n_obs) > 0).float()
    s = diam.Sampler(diam.make_config(d, P, 2, "fp32", beta=0.05, seed=3), None, None, rn(P, d).contiguous(), A=A, y=y,
                     prior_var=10.0)
    s.step_batch(1, rn(1, P, d), torch.full((1, P), 0.5 * 2.0 ** -52, dtype=torch.float64, device="cuda"))
    acc = s.get(diam.F_ACC).bool()
    x = s.get_f64(diam.F_X, (P, d))
    lp = s.get_f64(diam.F_LOGP, (P,))
    xf = x.float().double()
    t = A.double() @ xf.T
    ref = (y.double()[:, None] * t - torch.nn.functional.softplus(t)).sum(0) - 0.05 * (x * x).sum(1)
    u32 = 2.0 ** -24
    tol = ((d + 4) * u32 * (A.double().abs() @ xf.abs().T) + 6 * u32 * (t.abs() + 1)).sum(0) + 1e-12 * ref.abs()
    assert bool(acc.any()) and bool(((lp - ref).abs() <= tol).all())


@pytest.mark.parametrize("tiles", [2, 4])
def test_grouped_target_tiles(tiles):
    """The grouped target's 64-row tiles at ragged dimensions and chain counts:
    a first window's log alpha against a separate FP32 sampler's (the same
    products; shape 32 x 4 sums them in four chains instead of two, within 2 d
    u32 |log pi|)."""
    dims, P, n = [1, 5, 31, 33, 64, 97, 130, 260], 34, 4
    g = torch.Generator("cuda").manual_seed(2)
    rn = lambda *s: torch.randn(*s, generator=g, dtype=torch.float64, device="cuda")
    mus, Rs, xs = [rn(d) for d in dims], [(torch.eye(d, device="cuda") + rn(d, d) / d).float() for d in dims], [
        rn(P, d) for d in dims]
    b = diam.Batch(diam.make_batch_config(len(dims), P, n, seed=4), mus, Rs, xs)
    b.set_tiles(tiles)
    assert b.window()[0] in (diam.OK, diam.E_NOT_PD)
    for k, d in enumerate(dims):
        s = diam.Sampler(diam.make_config(d, P, n, "fp32"), mus[k], Rs[k], xs[k])
        ld = (d + 3) // 4 * 4
        W = b.get(k, diam.F_W).view(torch.float32).reshape(n, P, ld)[:, :, :d].double().contiguous()
        s.step_batch(n, W, b.get_f64(k, diam.F_U, (n, P)).contiguous())
        la_b, la_s = b.get_f64(k, diam.F_LA, (n, P)), s.get_f64(diam.F_LA, (n, P))
        if tiles == 2:
            assert torch.equal(la_b, la_s), d
        else:  # the first step: same states on both sides
            y = (xs[k] - mus[k]) @ Rs[k].double().T
            tol = 2 * d * 2.0 ** -24 * (100.0 + 4.0 * (y * y).sum(1))
            assert bool(((la_b[0] - la_s[0]).abs() <= tol).all()), d


@pytest.mark.parametrize("proposal", ["diam", "am"])
@pytest.mark.parametrize("prec,d,P,nproj,n_obs", [("fp64", 194, 5, 0, 0), ("fp64", 256, 3, 4, 0), ("fp64", 770, 66, 1, 0),
                                                  ("fp32", 2, 1, 1, 0), ("fp32", 34, 7, 4, 0), ("fp32", 130, 64, 0, 0),
                                                  ("fp32", 1154, 29, 2, 0), ("mixed", 64, 9, 2, 0),
                                                  ("mixed", 226, 50, 0, 0), ("mixed", 750, 31, 3, 0),
                                                  ("fp32", 128, 1024 * 4 + 1, 0, 0), ("fp32", 200, 6, 2, 300),
                                                  ("fp32", 62, 5, 0, 2000)])
def test_latency_bound_steps(prec, d, P, nproj, n_obs, proposal):
    """Steps that accept and propose at once (all of a call but its ends) give
    the bits of calls of one step each, which never do.  From these states the
    contracting proposals are nearly all accepted, the random walk's about half."""
    n = 6
    outs = []
    for split in (False, True):
        if n_obs:
            g = torch.Generator("cuda").manual_seed(d)
            rn = lambda *sh: torch.randn(*sh, generator=g, dtype=torch.float64, device="cuda")
            A, y = rn(n_obs, d).float(), (rn(n_obs) > 0).float()
            s = diam.Sampler(diam.make_config(d, P, n, prec, beta=0.25, seed=3, proposal=proposal), None, None,
                             (0.1 * rn(P, d)).contiguous(), A=A, y=y, prior_var=2.0)
        else:
            s, _, _, rn = sampler(prec, d, P, n, 5 + d, beta=0.25, proposal=proposal)
        trace = torch.zeros(n, 1 + nproj, P, dtype=torch.float64, device="cuda")
        s.set_trace(rn(nproj, d) if nproj else None, trace)
        W = (0.5 / np.sqrt(d) * rn(n, P, d)).contiguous()
        U = torch.linspace(0.05, 0.95, n * P, dtype=torch.float64, device="cuda").flip(0).reshape(n, P).contiguous()
        cnt = torch.zeros(P, dtype=torch.int32, device="cuda")
        la = []
        for t in range(n) if split else [slice(0, n)]:
            m = 1 if split else n
            s.step_batch(m, W[t].clone(), U[t].clone(), cnt)
            la.append(s.get(diam.F_LA).view(torch.float64)[:m * P].clone())
        outs.append([torch.cat(la), cnt, trace, s.get_f64(diam.F_X, (P, d)), s.get_f64(diam.F_Z, (P, d)),
                     s.get_f64(diam.F_LOGP, (P,))])
    for a, b in zip(*outs):
        assert torch.equal(a, b)
    assert proposal == "diam" or P == 1 or 0 < int(outs[0][1].sum()) < n * P
