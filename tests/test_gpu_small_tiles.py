"""The small tiles of the scan against the plan's own 512 x 128 tiles: every
accumulator takes the same matrix-core steps in the same order, so a test's
outputs have to be the same bits whichever tile computed them.

A scan of 32,768 markers x 512 phenotypes fills 256 CUs with 512 x 128 tiles
and takes those.  Short marker ranges of it, and panels of its first columns,
leave CUs idle there and take the small tiles (of 1 to 4 column blocks, with
and without Q^T g formed beside the tests)."""
import numpy as np
import pytest
import torch

from tests.gpu_common import lib, say

pytestmark = pytest.mark.gpu

M, P = 32768, 512
# marker ranges: one tile and less, edges of 128- and 256-row tiles, several rounds
RANGES = [(0, 1), (0, 127), (512, 641), (1024, 1535), (0, 4096), (2048, 10753), (0, M)]
# panels of the first columns: one phenotype, edges of one and two column blocks, more than two
WIDTHS = [1, 32, 33, 64, 65]


@pytest.fixture(scope="module")
def tgw():
    t = lib()
    t.init()
    return t


def _bits(outs):
    return {k: v.view(torch.int32) for k, v in outs.items()}


@pytest.mark.parametrize("precision,code,tile,n,k", [
    ("split8", "dosage", 0, 515, 10),   # nine chunks: a remainder after the first eight
    ("split8", "plink", 1, 1030, 3),    # 17 chunks; the order of tile 1's FP8 steps
    ("split8", "dosage", 6, 512, 10),   # exactly eight chunks; tile 6
    ("split8", "dosage", 0, 130, 20),   # three chunks, two covariate blocks
    ("split8", "dosage8", 0, 515, 10),
    ("split16", "dosage", 0, 960, 20),  # fifteen chunks
    ("split16", "dosage8", 0, 130, 16),
    ("split", "plink", 0, 515, 15),     # q = 16: one full covariate block
    ("fp32", "dosage", 0, 322, 10),
    ("fp32", "dosage8", 0, 130, 31),
])
def test_small_tiles_equal_wide(tgw, precision, code, tile, n, k):
    say(f"case: small tiles {precision} {code} tile={tile} n={n} k={k}")
    g = torch.Generator(device="cuda").manual_seed(n + k)
    if code == "dosage8":
        geno = torch.randint(0, 256, (M, (n + 63) // 64 * 64), generator=g, device="cuda", dtype=torch.uint8)
    else:
        geno = torch.randint(0, 256, (M, (n + 63) // 64 * 16), generator=g, device="cuda", dtype=torch.uint8)
    if k > 1:
        geno[7] = 0  # monomorphic (PLINK and dosage coding alike)
    C = torch.randn((k, n), generator=g, device="cuda", dtype=torch.float64).t()
    Y = torch.randn((P, n), generator=g, device="cuda").t()
    codes = {"dosage": tgw.CODE_DOSAGE, "plink": tgw.CODE_PLINK_BED, "dosage8": tgw.CODE_DOSAGE8}
    cov = tgw.fit_covariates(C)
    plan = tgw.Plan([tgw.prepare_phenotypes(cov, Y, precision)], tile=tile)
    want = _bits(tgw.scan(plan, geno, code=codes[code])[0])
    plan.check()
    assert torch.isfinite(want["r"].view(torch.float32)[8:]).float().mean() > 0.9
    narrow = [tgw.Plan([tgw.prepare_phenotypes(cov, Y[:, :p], precision)], tile=tile) for p in WIDTHS]
    for a, b in RANGES:
        for p, pl in zip([P] + WIDTHS, [plan] + narrow):
            got = tgw.make_outputs([p], b - a)
            for v in got[0].values():
                v.fill_(7.0)
            pl.scan(geno, got, a, b, codes[code])
            pl.check()
            for name, v in _bits(got[0]).items():
                assert torch.equal(v, want[name][a:b, :p]), f"{name}: range {a}..{b}, {p} columns"
    say(f"{len(RANGES) * (1 + len(WIDTHS))} scans equal the 512 x 128 tiles' bits")


def test_small_tiles_reduced_outputs(tgw):
    """Best test, top k and hit list of narrow panels, several in one plan with
    different covariates, equal those of the panels' dense outputs."""
    n, m = 700, 3000
    g = torch.Generator(device="cuda").manual_seed(5)
    geno = torch.randint(0, 256, (m, (n + 63) // 64 * 16), generator=g, device="cuda", dtype=torch.uint8)
    panels = []
    for p, k in ((40, 3), (1, 18), (33, 10)):
        C = torch.randn((k, n), generator=g, device="cuda", dtype=torch.float64).t()
        Y = torch.randn((p, n), generator=g, device="cuda").t()
        panels.append(tgw.prepare_phenotypes(tgw.fit_covariates(C), Y, "split8"))
    sizes = [pn.n_pheno for pn in panels]
    for group in ([0], [1], [2], [0, 1, 2]):
        sel = [panels[j] for j in group]
        plan = tgw.Plan(sel)
        dense = tgw.scan(plan, geno)
        best, top = tgw.make_best([sizes[j] for j in group]), tgw.make_topk([sizes[j] for j in group], 5)
        hits, count = tgw.make_hits(1 << 16)
        plan.set_hits(hits, count, 3.0)
        plan.scan(geno, [{"best": b, "topk": t} for b, t in zip(best, top)])
        plan.check()
        found = tgw.read_hits(hits, count)
        total = 0
        for i, o in enumerate(dense):
            nl, marker = tgw.unpack_best(best[i])
            t_abs = o["t"].abs().nan_to_num(-1.0)
            val, arg = t_abs.max(dim=0)
            np.testing.assert_array_equal(marker, arg.cpu().numpy())
            np.testing.assert_array_equal(nl, o["nlog10p"].gather(0, arg[None])[0].cpu().numpy())
            words = top[i].cpu().numpy().view("uint64")
            top_t = (words >> 32).astype("uint32").view("float32")
            np.testing.assert_array_equal(top_t, t_abs.topk(5, dim=0)[0].t().cpu().numpy())
            total += int((o["nlog10p"] >= 3.0).sum())
        assert found["count"] == total
        say(f"panels {group}: {total} hits, best and top 5 equal the dense outputs")
