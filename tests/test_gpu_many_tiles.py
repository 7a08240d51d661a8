"""A marker block of more than 2^24 small tiles, more than one launch can hold."""
import numpy as np
import pytest
import torch

from tests.gpu_common import lib, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["split8", "fp32"])
def test_more_tiles_than_a_launch_holds(precision):
    tgw = lib()
    tgw.init()
    n, m, p = 100, 1 << 20, 65_600
    say(f"case: many tiles {precision} n={n} m={m} p={p}")
    g = torch.Generator(device="cuda").manual_seed(1)
    geno = torch.randint(0, 256, (m, 32), generator=g, device="cuda", dtype=torch.uint8)
    Y = torch.randn((p, n), generator=g, device="cuda")
    # phenotypes that are a marker's calls but for a little noise: the only tests below 1e-40
    pairs = [(0, 0), (m - 1, p - 1), (127, 33), (128, 64_000), (524_287, 12_345), (524_288, 40_000), (1_000_000, 31)]
    for marker, pheno in pairs:
        codes = ((geno[marker, :25, None] >> torch.tensor([0, 2, 4, 6], device="cuda", dtype=torch.uint8)) & 3).flatten()
        calls = codes.float()
        calls[codes == 3] = calls[codes != 3].mean()
        Y[pheno] = calls + 1e-3 * Y[pheno]
    panel = tgw.prepare_phenotypes(tgw.fit_covariates(None, n_samples=n), Y.t(), precision)
    plan = tgw.Plan([panel])
    assert plan.info()["block_markers"] >= m
    plan.debug_set_path(1)  # 128 x 32
    assert m // 128 * ((p + 31) // 32) > 1 << 24
    hits, count = tgw.make_hits(1024)
    plan.set_hits(hits, count, 40.0)
    plan.scan(geno, [{}])
    plan.check()
    found = tgw.read_hits(hits, count)
    assert found["count"] == len(pairs)
    got = sorted(zip(np.asarray(found["marker"]).tolist(), np.asarray(found["pheno"]).tolist()))
    assert got == sorted(pairs)
