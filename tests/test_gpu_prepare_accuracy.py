"""The residual norm of a phenotype whose first sample is far off the others and
whose covariates explain nearly all of it: the standard errors say how good it is."""
import pytest
import torch

from tests.gpu_common import lib, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tgw():
    t = lib()
    t.init()
    return t


@pytest.mark.parametrize("spike", [1e3, 1e4])
def test_first_sample_far_off(tgw, spike):
    n, m, p = 2_000_003, 64, 16
    say(f"case: outlying first sample {spike}")
    g = torch.Generator(device="cuda").manual_seed(int(spike))
    c = torch.randn(n, generator=g, device="cuda", dtype=torch.float64)
    c[0] = spike
    Y = torch.randn((p, n), generator=g, device="cuda", dtype=torch.float64)
    # column 0 is noise; of the others the covariate leaves 1.4e-4 of the variance
    scale = 2.0 * (1 + torch.arange(p, device="cuda", dtype=torch.float64))
    noise = (1.4e-4 * c.var()).sqrt()
    Y[1:] = scale[1:, None] * (c + noise * Y[1:])
    geno = torch.randint(0, 256, (m, (n + 63) // 64 * 16), generator=g, device="cuda", dtype=torch.uint8)
    cov = tgw.fit_covariates(c[:, None])
    plan = tgw.Plan([tgw.prepare_phenotypes(cov, Y.t(), "split16")])
    out = tgw.scan(plan, geno)[0]
    plan.check()
    c -= c.mean()
    c /= c.norm()
    Y -= Y.mean(dim=1, keepdim=True)
    for _ in range(2):
        Y -= (Y @ c)[:, None] * c
    s = Y.norm(dim=1)
    assert (s[1:] / scale[1:] / n ** 0.5 / noise - 1).abs().max() < 0.01
    # SE = s_p sqrt(1 - r^2) times the same factor in a marker's whole row: against column 0, s_p's FP32
    # rounding (6e-8 both) and the mean over 64 markers of four more roundings each, 6e-8 / 8
    r2 = out["r"].double().square()
    se = (out["se"].double() / torch.sqrt(1 - r2))
    got = (se / se[:, :1]).mean(dim=0)
    err = (got / (s / s[0]) - 1).abs().max().item()
    say(f"largest error of ||y_res|| {err:.2e}")
    assert err < 3e-7
