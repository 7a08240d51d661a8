"""Phenotype preparation at the edges of its tiles (16 columns, 16-slot tiles
of the covariate basis, segments of samples) and on columns that need care
(offsets, degenerate columns, columns that the covariates nearly explain):
what a scan with the prepared panel gives, against the FP64 oracle."""
import numpy as np
import pytest
import torch

from synth import pack_codes_np, row_bytes_for
from tests.gpu_common import compare, lib, oracle_scan, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tgw():
    t = lib()
    t.init()
    return t


@pytest.mark.parametrize("n,p,k,precision,y64,pad", [
    (4033, 1, 0, "split8", False, 0),    # 64 chunks, the last with one sample; intercept only
    (4096, 15, 3, "split", True, 0),     # whole chunks
    (4097, 16, 15, "split16", False, 3), # q = 16: one full slot tile; a column stride of n + 3
    (5003, 17, 16, "fp32", True, 0),     # q = 17: two slot tiles
    (6000, 33, 31, "split8", True, 1),   # every slot
    (9001, 48, 10, "split8", False, 0),
])
def test_prepare_edges(tgw, n, p, k, precision, y64, pad):
    say(f"case: prepare n={n} p={p} k={k} {precision} fp64={y64} pad={pad}")
    rng = np.random.default_rng(n + p)
    m = 40
    codes = rng.binomial(2, rng.uniform(0.05, 0.5, m)[:, None], size=(m, n)).astype(np.uint8)
    codes[rng.random((m, n)) < 0.01] = 3
    C = rng.standard_normal((n, k))
    Y = rng.standard_normal((n, p)) + 0.2 * (codes[3][:, None] == 1)
    if k:
        Y += C @ rng.standard_normal((k, p))
    Y[:, p // 2] = 1e4 + Y[:, p // 2]                     # an offset far above the spread
    if p > 4:
        Y[:, 0] = 3.25                                     # constant: degenerate
        Y[0, 1] = 500.0                                    # the first sample is an outlier
        if k:
            Y[:, 2] = C[:, 0] + 1e-4 * rng.standard_normal(n)  # nearly explained by a covariate
    Y = Y.astype(np.float64 if y64 else np.float32)
    ref = oracle_scan(codes, C, Y.astype(np.float64))
    buf = torch.zeros((p, n + pad), dtype=torch.float64 if y64 else torch.float32, device="cuda")
    buf[:, :n] = torch.from_numpy(np.ascontiguousarray(Y.T)).cuda()
    cov = tgw.fit_covariates(torch.from_numpy(C).cuda() if k else None, n_samples=n)
    panel = tgw.prepare_phenotypes(cov, buf.t()[:n], precision)
    plan = tgw.Plan([panel])
    out = tgw.scan(plan, torch.from_numpy(pack_codes_np(codes, row_bytes_for(n))).cuda())[0]
    plan.check()
    got = {name: v.cpu().numpy() for name, v in out.items()}
    if p > 4:
        assert np.isnan(got["r"][:, 0]).all() and np.isnan(ref["r"][:, 0]).all()
    compare(got, ref, ref["df"], f"prepare n={n} p={p} k={k} ")


@pytest.mark.parametrize("y64", [False, True])
@pytest.mark.parametrize("row,value", [(0, np.nan), (4999, np.inf)])
def test_prepare_rejects_nonfinite(tgw, y64, row, value):
    n, p = 5000, 20
    Y = np.random.default_rng(3).standard_normal((n, p))
    Y[row, 17] = value
    cov = tgw.fit_covariates(None, n_samples=n)
    with pytest.raises(tgw.TgwError) as e:
        tgw.prepare_phenotypes(cov, torch.from_numpy(Y).cuda().to(torch.float64 if y64 else torch.float32), "split8")
    assert e.value.status == tgw.ERR_NONFINITE


def test_prepare_without_room_for_scratch(tgw):
    """An arena that holds the panel but not the preparation's scratch: the
    panel is prepared all the same, with the same outputs to FP32 rounding."""
    n, p, m = 6000, 64, 30
    rng = np.random.default_rng(11)
    codes = rng.binomial(2, 0.3, size=(m, n)).astype(np.uint8)
    Y = torch.from_numpy(rng.standard_normal((p, n)).astype(np.float32)).cuda().t()
    geno = torch.from_numpy(pack_codes_np(codes, row_bytes_for(n))).cuda()
    cov = tgw.fit_covariates(None, n_samples=n)

    def prepared():
        panel = tgw.prepare_phenotypes(cov, Y, "split16")
        return panel, tgw.scan(tgw.Plan([panel], block_markers=512, tail_capacity=1024), geno)[0]

    _, want = prepared()
    arena = tgw.torch_arena(64 << 20)
    arena.register()
    try:
        big = prepared()
        need = arena.info().peak
        del big
        in_use = arena.info().in_use
    finally:
        tgw.set_allocator()
    arena.close()
    assert in_use == 0
    op = (n + 63) // 64 * 64 * p * 4
    small = tgw.torch_arena(op + (200 << 10))  # the operand, the table and the per-column constants
    assert small.info().capacity < need
    small.register()
    try:
        panel = tgw.prepare_phenotypes(cov, Y, "split16")
    finally:
        tgw.set_allocator()
    assert small.info().n_failed >= 1
    got = tgw.scan(tgw.Plan([panel]), geno)[0]
    for name in want:
        torch.testing.assert_close(got[name], want[name], rtol=1e-6, atol=1e-9, equal_nan=True)
    del panel
    small.close()
