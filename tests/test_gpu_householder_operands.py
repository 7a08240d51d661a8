"""Covariates so ill-conditioned that their basis comes from Householder
reflections: a scan adjusts for the same space as with a well-conditioned basis
of it."""
import pytest
import torch

from tests.gpu_common import lib, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tgw():
    t = lib()
    t.init()
    return t


@pytest.mark.parametrize("precision", ["split8", "split", "fp32"])
@pytest.mark.parametrize("n,k", [(70, 2), (1000, 15), (4097, 16), (5003, 31)])
def test_same_space_same_scan(tgw, precision, n, k):
    say(f"case: Householder operands n={n} k={k} {precision}")
    g = torch.Generator(device="cuda").manual_seed(n)
    geno = torch.randint(0, 256, (300, (n + 63) // 64 * 16), generator=g, device="cuda", dtype=torch.uint8)
    C = torch.randn((k, n), generator=g, device="cuda", dtype=torch.float64)
    Y = (torch.randn((40, n), generator=g, device="cuda", dtype=torch.float64) + C[-1]).t()
    ill = C.clone()
    ill[-1] = C[0] + 1e-6 * C[-1]
    outs = []
    for X in (C, ill):
        plan = tgw.Plan([tgw.prepare_phenotypes(tgw.fit_covariates(X.t()), Y, precision)])
        outs.append(tgw.scan(plan, geno)[0])
        plan.check()
    # the last column of the ill-conditioned basis is good to 1e-16 / 1e-6; r to the rounding of the operands
    for name, tol in (("r", 1e-5), ("nlog10p", 1e-4)):
        a, b = outs[0][name], outs[1][name]
        assert torch.isfinite(a).all()
        assert ((a - b).abs() <= tol * torch.clamp(a.abs(), min=1.0)).all(), name
