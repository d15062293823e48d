"""Local updates (M > 1) in which some chains' factorisations fail: the failed
chain keeps its pair, the others adopt theirs, before and after updates that
exchanged all pairs at once."""
import numpy as np
import pytest
import torch

from paper_1506_05741_amd import diam

pytestmark = pytest.mark.gpu

U64 = 2.0 ** -53


@pytest.mark.parametrize("tries", [0, 13])
@pytest.mark.parametrize("d,P,bad", [(8, 5, 1), (70, 3, 2), (129, 18, 0)])
def test_failed_chain_keeps_its_pair(d, P, bad, tries):
    """Two updates in which every chain succeeds, then two in which one chain's
    covariance has lost its small eigenvalues: that chain jumped by 1e10, so the
    rounding of its second moments, 1e20 u, is far above them.  Without retries
    it keeps its pair; with them it gets the pair of a jittered covariance."""
    n = 4
    g = torch.Generator("cuda").manual_seed(d)
    rn = lambda *s: torch.randn(*s, generator=g, dtype=torch.float64, device="cuda")
    R = 1e-13 * torch.eye(d, dtype=torch.float64, device="cuda")  # nearly flat: the jump is accepted
    s = diam.Sampler(diam.make_config(d, P, n, "fp64", beta=0.3, seed=7, M=6, jitter_tries=tries),
                     torch.zeros(d, dtype=torch.float64, device="cuda"), R, rn(P, d).contiguous())
    assert s.seed_moments(torch.eye(d, dtype=torch.float64, device="cuda"),
                          torch.zeros(d, dtype=torch.float64, device="cuda"), 50.0)[0] == diam.OK
    fields = lambda: [s.get_f64(diam.F_LP, (P, d, d)).clone(), s.get_f64(diam.F_XREFP, (P, d)).clone(),
                      s.get_f64(diam.F_Z, (P, d)).clone(), s.get_f64(diam.F_ZQ, (P,)).clone()]
    for update in range(4):
        W = rn(n, P, d)
        if update == 2:
            W[0, bad] *= 1e10
        U = torch.full((n, P), 0.5, dtype=torch.float64, device="cuda")
        U[0] = 1e-300
        s.step_batch(n, W.contiguous(), U)
        s.merge_moments()
        before, X = fields(), s.get_f64(diam.F_X, (P, d)).clone()
        assert update < 2 or float(X[bad].abs().max()) > 1e8
        fails = update >= 2 and tries == 0
        status, jitter = s.update_proposal()
        assert status == (diam.E_NOT_PD if fails else diam.OK) and (jitter >= 0) == (update >= 2)
        after = fields()
        for p in range(P):
            if fails and p == bad:
                assert all(torch.equal(a[p], b[p]) for a, b in zip(after, before))
                continue
            L, xr, z = torch.tril(after[0][p].T), after[1][p], after[2][p]
            assert not torch.equal(after[0][p], before[0][p]) and not torch.equal(xr, before[1][p])
            res, m = L @ z - (X[p] - xr), L.abs() @ z.abs() + X[p].abs() + xr.abs()
            assert bool((res.abs() <= 8 * (d + 8) * U64 * m).all())
            assert abs(float(after[3][p] - (z * z).sum())) <= (d + 8) * U64 * float(after[3][p])
