"""Which kernels a call launches, from the profiler's records, where a rule on
sizes chooses among kernels: each side of the rule's line."""
import numpy as np
import pytest
import torch
from torch.profiler import ProfilerActivity, profile

from paper_1506_05741_amd import diam

pytestmark = pytest.mark.gpu


def kernels(call):
    """Names of the kernels that `call` launches."""
    call()
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        call()
        torch.cuda.synchronize()
    return [e.name for e in p.events() if "dk::" in e.name]


def sampler(prec, d, P, n_lag, **kw):
    g = torch.Generator("cuda").manual_seed(d + P)
    rn = lambda *s: torch.randn(*s, generator=g, dtype=torch.float64, device="cuda")
    R = torch.eye(d, dtype=torch.float64, device="cuda") + rn(d, d) / np.sqrt(d)
    if prec != "fp64":
        R = R.float()
    return diam.Sampler(diam.make_config(d, P, n_lag, prec, seed=3, beta=0.3, **kw), rn(d), R.contiguous(),
                        rn(P, d).contiguous())


@pytest.mark.parametrize("d,P,n,one", [(64, 64, 1, True), (64, 700, 1, True), (64, 2048, 2, False), (64, 2048, 3, True),
                                       (32, 16384, 23, False), (32, 16384, 24, True), (128, 64, 1, True),
                                       (128, 256, 2, False), (128, 256, 3, True), (100, 8192, 81, False),
                                       (100, 8192, 82, True), (100, 8193, 82, False), (192, 64, 1, True),
                                       (192, 256, 6, False), (192, 256, 7, True), (192, 1024, 25, False),
                                       (192, 1024, 26, True), (193, 4, 8, False)])
def test_steps_in_one_launch_only_where_a_call_earns_it_back(d, P, n, one):
    """The loop with R in registers reads R once per chain and call: a call of
    few steps of many chains takes the launches per step (d = 128, 8192 chains,
    one step: 511 us in the loop, 44 in launches)."""
    names = kernels(lambda s=sampler("fp64", d, P, 2 * n): s.step_batch(n))
    assert any("k_steps_resident" in k for k in names) == one


@pytest.mark.parametrize("prec,d,P,kernel", [("fp64", 64, 8192, "k_tgt_gauss_t<32>"), ("fp64", 200, 300, "k_tgt_split<double>"),
                                             ("fp64", 1024, 192, "k_tgt_split<double>"),
                                             ("fp64", 1024, 256, "k_tgt_gauss_t<32>"),
                                             ("fp64", 2048, 512, "k_tgt_gauss_t<64>"),
                                             ("fp64", 129, 2048, "k_tgt_gauss<double"),
                                             ("fp64", 129, 1024, "k_tgt_split<double>"),
                                             ("fp32", 64, 2048, "k_tgt_split<float>"),
                                             ("fp32", 64, 8192, "k_tgt_gauss<float"),
                                             ("fp32", 1024, 512, "k_tgt_split<float>"),
                                             ("fp32", 1024, 768, "k_tgt_gauss<float"),
                                             ("fp32", 700, 1024, "k_tgt_split<float>"),
                                             ("mixed", 64, 8192, "k_tgt_gauss<float")])
def test_target_kernel_by_size(prec, d, P, kernel):
    """The split target kernel's time grows with its workgroups, the tile
    kernels take that of one tile: many chains of a small dimension belong to
    the latter (d = 64, 8192 chains: FP32 12.4 us split, 6.3 tiled)."""
    names = kernels(lambda s=sampler(prec, d, P, 4): s.step_batch(2))
    assert any(kernel in k for k in names) and sum("k_tgt" in k for k in names) == 2


@pytest.mark.parametrize("d,P", [(2, 1100), (14, 1041), (34, 1025), (62, 3000), (66, 1500), (130, 607), (254, 531)])
def test_engine_target_of_few_dimensions_and_many_chains(d, P):
    """The FP64 engine's 32 x 32 tiles with less than one to a few slices of K,
    against FP64 products (a sum of d + 8 terms, 8 (d + 8) u)."""
    g = torch.Generator("cuda").manual_seed(d)
    rn = lambda *s: torch.randn(*s, generator=g, dtype=torch.float64, device="cuda")
    R, mu, x0 = torch.eye(d, dtype=torch.float64, device="cuda") + rn(d, d) / np.sqrt(d), rn(d), rn(P, d)
    s = diam.Sampler(diam.make_config(d, P, 4, "fp64", beta=0.05, seed=5), mu, R, x0)
    W, U = 0.2 * rn(1, P, d), torch.full((1, P), 0.5 * 2.0 ** -52, dtype=torch.float64, device="cuda")
    names = kernels(lambda: s.step_batch(1, W, U))
    assert any("k_tgt_gauss_t<32>" in k for k in names)
    assert bool(s.get(diam.F_ACC).bool().all())  # accepted unless log alpha < -36
    y = (s.get_f64(diam.F_X, (P, d)) - mu) @ R.T
    ref = -0.5 * (y * y).sum(1)
    assert bool(((s.get_f64(diam.F_LOGP, (P,)) - ref).abs() <= 8 * (d + 8) * 2.0 ** -53 * ref.abs()).all())


@pytest.mark.parametrize("tiles", [2, 4])
@pytest.mark.parametrize("dims,P,engine", [([320, 64, 33], 32, (False, False)), ([256, 230, 7], 64, (False, False)),
                                           ([300, 310], 32, (True, False)), ([200, 130, 33], 20, (True, False)),
                                           ([128, 64], 32, (False, True)), ([192] * 132, 32, (False, True)),
                                           ([192] * 132 + [65], 32, (True, True)), ([190] * 70, 24, (True, True))])
def test_grouped_target_kernel_by_problem_set(dims, P, engine, tiles):
    """Few tiles, or none at an edge, belong to the tile kernels (one problem
    of 1024: 9.2 us against the engine's 18.6 in shape 32 x 4).  Both give the
    log ratios of a separate FP32 sampler: shape 64 x 2 the same bits, 32 x 4,
    whose four chains of a sum are added in another order, within 2 d u32 of
    the squares summed."""
    n = 2
    g = torch.Generator("cuda").manual_seed(3)
    rn = lambda *s: torch.randn(*s, generator=g, dtype=torch.float64, device="cuda")
    mus, xs = [rn(d) for d in dims], [rn(P, d) for d in dims]
    Rs = [(torch.eye(d, device="cuda") + rn(d, d) / d).float() for d in dims]
    b = diam.Batch(diam.make_batch_config(len(dims), P, n, seed=4), mus, Rs, xs)
    b.set_graph(False)
    b.set_tiles(tiles)
    first = [None]

    def window():
        b.window()
        if first[0] is None:
            first[0] = [(b.get(k, diam.F_W).clone(), b.get_f64(k, diam.F_U, (n, P)).clone(),
                         b.get_f64(k, diam.F_LA, (n, P)).clone()) for k in range(len(dims))]

    names = kernels(window)
    assert any("gk_tgt_t<" in k for k in names) == engine[tiles == 4]
    for k in range(len(dims))[-6:]:
        d, (W, U, la) = dims[k], first[0][k]
        s = diam.Sampler(diam.make_config(d, P, n, "fp32"), mus[k], Rs[k], xs[k])
        ld = (d + 3) // 4 * 4
        s.step_batch(n, W.view(torch.float32).reshape(n, P, ld)[:, :, :d].double().contiguous(), U.contiguous())
        ref = s.get_f64(diam.F_LA, (n, P))
        if tiles == 2:
            assert torch.equal(la, ref), d
        else:  # the first step: same states on both sides
            y = (xs[k] - mus[k]) @ Rs[k].double().T
            assert bool(((la[0] - ref[0]).abs() <= 2 * d * 2.0 ** -24 * (100.0 + 4.0 * (y * y).sum(1))).all()), d


@pytest.mark.parametrize("n_obs,d,P,engine", [(64, 256, 64, False), (128, 300, 128, False), (16384, 256, 128, False),
                                              (16448, 256, 128, True), (63, 256, 64, True), (128, 256, 63, True),
                                              (128, 252, 64, True), (128, 301, 64, False), (129, 301, 63, False)])
def test_logistic_kernel_by_size(n_obs, d, P, engine):
    """Few whole tiles belong to the tile kernel (2048 dimensions, 16000
    observations, 64 chains: 65 us a step, 74 on the engine), unaligned rows
    too.  Against FP64 at the accepted states: an FP32 dot product of d terms
    errs by (d + 4) u32 sum |a x|, a term's evaluation by 6 u32 (|t| + 1)."""
    g = torch.Generator("cuda").manual_seed(n_obs + d)
    rn = lambda *s: torch.randn(*s, generator=g, dtype=torch.float64, device="cuda")
    A, y = (rn(n_obs, d) / np.sqrt(d)).float(), (rn(n_obs) > 0).float()
    s = diam.Sampler(diam.make_config(d, P, 8, "fp32", beta=0.05, seed=3), None, None, rn(P, d).contiguous(), A=A, y=y,
                     prior_var=10.0)
    W, U = 0.2 * rn(1, P, d), torch.full((1, P), 0.5 * 2.0 ** -52, dtype=torch.float64, device="cuda")
    names = kernels(lambda: s.step_batch(1, W, U))
    assert any("k_tgt_logreg_t" in k for k in names) == engine
    assert bool(s.get(diam.F_ACC).bool().all())  # accepted unless log alpha < -36
    x = s.get_f64(diam.F_X, (P, d))
    xf = x.float().double()
    t = A.double() @ xf.T
    ref = (y.double()[:, None] * t - torch.nn.functional.softplus(t)).sum(0) - 0.05 * (x * x).sum(1)
    u32 = 2.0 ** -24
    tol = ((d + 4) * u32 * (A.double().abs() @ xf.abs().T) + 6 * u32 * (t.abs() + 1)).sum(0) + 1e-12 * ref.abs()
    assert bool(((s.get_f64(diam.F_LOGP, (P,)) - ref).abs() <= tol).all())


def test_merge_of_one_tile_and_many_splits():
    """The sum over the splits of the scatter has its loads in flight together
    (d = 64, 64 splits on one workgroup: 39 us, 89 with one load at a time,
    beside a scatter of 37)."""
    s = sampler("mixed", 64, 8192, 16)

    def window():
        s.step_batch(16)
        s.merge_moments()

    window()
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        for _ in range(5):
            window()
        torch.cuda.synchronize()
    us = lambda name: min(e.device_time for e in p.events() if name in e.name)
    assert us("k_merge") < 1.6 * us("k_syrk")


@pytest.mark.parametrize("proposal", ["diam", "am"])
@pytest.mark.parametrize("d,P,cuts", [(64, 2048, (8, 1, 4, 2, 2, 3)), (101, 300, (2, 9, 1, 5)), (192, 256, (7, 3, 8))])
def test_window_cut_into_calls_of_both_kinds(d, P, cuts, proposal):
    """Calls that run in one launch and calls that launch per step take over
    from each other: decisions, states, log densities and the window's mean
    against the recursion in FP64 on the directions each call drew (t steps err
    by at most t times a step's 4 u, log pi by 8 (d + n) u of its terms)."""
    n, beta, U64 = sum(cuts), 0.25, 2.0 ** -53
    g = torch.Generator("cuda").manual_seed(d)
    rn = lambda *sh: torch.randn(*sh, generator=g, dtype=torch.float64, device="cuda")
    R, mu = torch.eye(d, dtype=torch.float64, device="cuda") + rn(d, d) / np.sqrt(d), rn(d)
    s = diam.Sampler(diam.make_config(d, P, n, "fp64", seed=1, beta=beta, proposal=proposal), mu, R.contiguous(),
                     rn(P, d).contiguous())
    rho = 1.0 if proposal == "am" else np.sqrt(1 - beta * beta)
    x, z, xr = s.get_f64(diam.F_X, (P, d)).clone(), s.get_f64(diam.F_Z, (P, d)).clone(), s.get_f64(diam.F_XREF, (d,))
    lp, tot, cnt = s.get_f64(diam.F_LOGP, (P,)).clone(), 0.0, torch.zeros(P, dtype=torch.int32, device="cuda")
    taken, kinds = torch.zeros_like(cnt), set()
    for m in cuts:
        W = (0.4 / np.sqrt(d) * rn(m, P, d)).contiguous()
        U = torch.rand(m, P, generator=g, dtype=torch.float64, device="cuda").clamp_(1e-12)
        with profile(activities=[ProfilerActivity.CUDA]) as p:
            s.step_batch(m, W, U, cnt)
            torch.cuda.synchronize()
        kinds.add(any("k_steps_resident" in e.name for e in p.events()))
        Xi = s.get(diam.F_XI).view(torch.float64)[:m * P * d].reshape(m, P, d)
        Acc = s.get(diam.F_ACC)[:m * P].reshape(m, P).bool()
        mag = torch.maximum(x.abs(), z.abs()).amax() + Xi.abs().amax() * m + mu.abs().amax()
        for t in range(m):
            xp, zp = xr + rho * (x - xr) + Xi[t], rho * z + beta * W[t]
            y = (xp - mu) @ R.T
            lpp = -0.5 * (y * y).sum(1)
            la = lpp - lp + (0.0 if proposal == "am" else 0.5 * ((zp * zp).sum(1) - (z * z).sum(1)))
            assert torch.equal(Acc[t], torch.log(U[t]) < la)
            x, z = torch.where(Acc[t][:, None], xp, x), torch.where(Acc[t][:, None], zp, z)
            lp, tot = torch.where(Acc[t], lpp, lp), tot + x.sum(0)
        taken += Acc.sum(0, dtype=torch.int32)
        assert bool(((s.get_f64(diam.F_X, (P, d)) - x).abs() <= 4 * n * U64 * mag).all())
        assert bool(((s.get_f64(diam.F_Z, (P, d)) - z).abs() <= 4 * n * U64 * mag).all())
        ya = mu.abs() @ R.abs().T + x.abs() @ R.abs().T
        assert bool(((s.get_f64(diam.F_LOGP, (P,)) - lp).abs() <= 8 * (d + n) * U64 * (ya * ya).sum(1)).all())
    assert kinds == {True, False} and torch.equal(cnt, taken)
    assert proposal == "diam" or 0 < int(taken.sum()) < n * P  # contracting proposals may all be accepted
    s.merge_moments()
    assert bool(((s.get_f64(diam.F_M, (d,)) - tot / (n * P)).abs() <= 4 * (n * P + n) * U64 * mag).all())
