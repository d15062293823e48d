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


@pytest.mark.parametrize("d,P,n,one", [(64, 64, 1, True), (64, 65, 1, True), (64, 2048, 1, False), (64, 2048, 2, True),
                                       (32, 16384, 8, False), (32, 16384, 16, True), (128, 64, 1, True),
                                       (128, 256, 1, False), (128, 256, 2, True), (100, 8192, 16, False),
                                       (100, 8192, 64, True), (100, 8193, 64, False), (192, 64, 1, True),
                                       (192, 256, 4, False), (192, 256, 6, True), (192, 1024, 16, False),
                                       (192, 1024, 24, True), (193, 4, 8, False)])
def test_steps_in_one_launch_only_where_a_call_earns_it_back(d, P, n, one):
    """The loop with R in registers reads R once per chain and call: a call of
    few steps of many chains takes the launches per step (d = 128, 8192 chains,
    one step: 511 us in the loop, 44 in launches)."""
    names = kernels(lambda s=sampler("fp64", d, P, 2 * n): s.step_batch(n))
    assert any("k_steps_resident" in k for k in names) == one
