"""Cohorts so long that a column of the covariate basis lies 4 GiB and more
behind its first element (31 covariates: from 17.3 million samples)."""
import pytest
import torch

from tests.gpu_common import lib, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tgw():
    t = lib()
    t.init()
    return t


def _pack(calls):
    m, n = calls.shape
    row = (n + 63) // 64 * 64
    out = torch.full((m, row), 3, dtype=torch.uint8, device="cuda")
    out[:, :n] = calls
    b = out.view(m, row // 4, 4)
    return (b[..., 0] | (b[..., 1] << 2) | (b[..., 2] << 4) | (b[..., 3] << 6)).contiguous()


@pytest.mark.parametrize("precision", ["split8", "fp32"])
def test_last_covariate_beyond_4_gib(tgw, precision):
    """The last covariate makes up most of both phenotypes and of marker 0
    (which so takes the FP64 path): its projections are what the preparation
    and that path have to take out."""
    n, k = 17_400_003, 31
    say(f"case: many samples n={n} k={k} {precision}")
    assert k * ((n + 63) // 64 * 64) * 8 >= 1 << 32
    g = torch.Generator(device="cuda").manual_seed(7)
    calls = (torch.rand((2, n), generator=g, device="cuda") < 0.4).to(torch.uint8)
    calls += torch.rand((2, n), generator=g, device="cuda") < 0.4
    C = torch.randn((k, n), generator=g, device="cuda", dtype=torch.float64)
    C[k - 1] = calls[0].double() + 0.4 * C[k - 1]
    Y = torch.randn((2, n), generator=g, device="cuda", dtype=torch.float64)
    Y[0] += 3.0 * C[k - 1]
    Y[1] += 0.01 * calls[0] + 0.01 * calls[1] - 2.0 * C[k - 1]

    cov = tgw.fit_covariates(C.t())
    panel = tgw.prepare_phenotypes(cov, Y.t(), precision)
    plan = tgw.Plan([panel], block_markers=512, tail_capacity=1024)
    out = tgw.scan(plan, _pack(calls))[0]
    plan.check()

    # residuals against [1 | C] by the normal equations (unit columns: condition about 10)
    Z = torch.cat([calls.double(), Y])
    C -= C.mean(dim=1, keepdim=True)
    Z -= Z.mean(dim=1, keepdim=True)
    for _ in range(2):
        B = torch.linalg.solve(C @ C.t(), C @ Z.t())
        Z -= B.t() @ C
    gr, yr = Z[:2], Z[2:]
    r = (gr @ yr.t()) / (gr.norm(dim=1)[:, None] * yr.norm(dim=1)[None])
    df = n - k - 2
    beta = r * yr.norm(dim=1)[None] / gr.norm(dim=1)[:, None]
    se = (yr.norm(dim=1)[None] / gr.norm(dim=1)[:, None]) * torch.sqrt((1 - r * r) / df)
    say(f"r {r.tolist()} got {out['r'].tolist()}")
    # the FP64 path contracts the stored operand: its rounding (relative 2^-16 per sample, of random sign) and
    # the FP32 outputs; the other marker: the bound on r of the matrix-core forms
    assert (out["r"].double() - r)[0].abs().max() < 1e-6
    assert (out["r"].double() - r)[1].abs().max() < 1e-5
    assert (out["se"].double() / se - 1).abs().max() < 2e-6
    assert ((out["beta"].double() - beta) / se)[0].abs().max() < 1e-6 * df ** 0.5
