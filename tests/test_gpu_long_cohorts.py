"""Cohorts of more than 65,536 samples: the FP16 forms add segments of the
samples up, side by side where a scan leaves CUs idle, else one after the other.
The segments and their order are those of the sample count alone, so a test's
outputs are the same bits whichever kernel computed them; up to 65,536 samples
there is one segment."""
import numpy as np
import pytest
import torch

from tests.gpu_common import lib, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tgw():
    t = lib()
    t.init()
    return t


def _bits(o):
    return {k: v.view(torch.int32) for k, v in o.items()}


def _oracle_r(geno, C, Y, rows, code):
    """Partial correlations of the given rows, in FP64 from the definition."""
    n = Y.shape[0]
    if code == "dosage8":
        g = geno[rows, :n].double()
        g[g == 255] = float("nan")
    else:
        b = geno[rows][:, :, None]
        g = ((b >> torch.tensor([0, 2, 4, 6], device="cuda", dtype=torch.uint8)) & 3).reshape(len(rows), -1)[:, :n]
        g = torch.tensor([0.0, 1.0, 2.0, float("nan")], device="cuda", dtype=torch.float64)[g.long()]
    mean = g.nanmean(dim=1, keepdim=True)
    g = torch.where(g.isnan(), mean, g)
    Q = torch.linalg.qr(torch.cat([torch.ones((n, 1), device="cuda", dtype=torch.float64), C], dim=1))[0]
    g = g - (g @ Q) @ Q.t().contiguous()
    y = Y.double()
    y = y - Q @ (Q.t().contiguous() @ y)
    return (g / g.norm(dim=1, keepdim=True)) @ (y / y.norm(dim=0, keepdim=True))


@pytest.mark.parametrize("precision,code,tile,n,m,k", [
    ("split8", "dosage", 0, 65_536, 32_768, 10),   # the most samples of one segment
    ("split8", "dosage", 0, 65_537, 32_768, 10),   # a second segment of one sample
    ("split8", "dosage", 1, 65_600 + 515, 32_768, 20),
    ("split8", "dosage", 6, 131_073, 16_384, 3),   # three segments, the last of one sample
    ("split8", "dosage8", 0, 65_537, 8192, 10),
    ("split16", "dosage", 2, 70_001, 32_768, 10),  # a tile without segments of its own
    ("split16", "dosage8", 2, 66_000, 8192, 20),
    ("split", "dosage", 0, 66_050, 32_768, 10),    # never segmented
    ("split8", "dosage", 0, 524_353, 4096, 10),    # longer segments, eight of them
    ("fp32", "dosage", 0, 66_050, 4096, 10),
])
def test_segments(tgw, precision, code, tile, n, m, k):
    say(f"case: segments {precision} {code} tile={tile} n={n} m={m} k={k}")
    p = 512
    g = torch.Generator(device="cuda").manual_seed(n + k)
    row = (n + 63) // 64 * (64 if code == "dosage8" else 16)
    geno = torch.randint(0, 256, (m, row), generator=g, device="cuda", dtype=torch.uint8)
    C = torch.randn((k, n), generator=g, device="cuda", dtype=torch.float64).t()
    Y = torch.randn((p, n), generator=g, device="cuda").t()
    c = {"dosage": tgw.CODE_DOSAGE, "dosage8": tgw.CODE_DOSAGE8}[code]
    cov = tgw.fit_covariates(C)
    panel = tgw.prepare_phenotypes(cov, Y, precision)
    plan = tgw.Plan([panel], tile=tile)
    want = tgw.scan(plan, geno, code=c)[0]
    plan.check()

    # a test's FP32 sums take under 4,096 matrix-core steps per segment, each
    # rounded to half an ulp of a partial sum of under about 4 sqrt(N) (in units
    # where r is the sum over N): 4096 * 2^-24 * 4 / sqrt(65536) = 4e-6 at the
    # most; the unsegmented forms take up to n / 2 steps with errors of random
    # signs, which stays under the same
    rows = list(range(0, m, m // 32))
    ref = _oracle_r(geno, C, Y, rows, code)
    err = (want["r"][rows].double() - ref).abs().max().item()
    say(f"largest error of r against FP64: {err:.2e}")
    assert err < 4e-6

    want = _bits(want)

    def same(outs, a, b, p_, what):
        for name, v in _bits(outs).items():
            assert torch.equal(v, want[name][a:b, :p_]), f"{name}: {what}"

    for width in (p, 1, 33, 65):
        pl = plan if width == p else tgw.Plan([tgw.prepare_phenotypes(cov, Y[:, :width], precision)], tile=tile)
        for a, b in ((0, 1), (512, 641), (1024, 1024 + m // 8)):
            got = tgw.make_outputs([width], b - a)
            pl.scan(geno, got, a, b, c)
            pl.check()
            same(got[0], a, b, width, f"range {a}..{b}, {width} columns")
    got = tgw.make_outputs([p], m)
    tgw.scan_static([panel], geno, got, code=c, tile=tile)
    torch.cuda.synchronize()
    same(got[0], 0, m, p, "without a plan")


def test_segments_in_little_memory(tgw):
    """A plan whose memory does not hold the segments of a whole round takes
    them in more and smaller steps, to the same bits."""
    n, m = 140_001, 1500
    g = torch.Generator(device="cuda").manual_seed(1)
    geno = torch.randint(0, 256, (m, (n + 63) // 64 * 16), generator=g, device="cuda", dtype=torch.uint8)
    cov = tgw.fit_covariates(torch.randn((5, n), generator=g, device="cuda", dtype=torch.float64).t())
    # Q^T g beside the tests, and on its own; one row of column tiles that is too long for the buffer
    for width in (1, 96, 1500):
        panel = tgw.prepare_phenotypes(cov, torch.randn((width, n), generator=g, device="cuda").t(), "split8")
        want = tgw.scan(tgw.Plan([panel], block_markers=1024, tail_capacity=1024), geno)[0]
        arena = tgw.torch_arena(4 << 20)
        arena.register()
        try:
            plan = tgw.Plan([panel], block_markers=1024, tail_capacity=1024)
        finally:
            tgw.set_allocator()
        assert arena.info().n_failed >= 1
        got = tgw.make_outputs([width], m)
        plan.scan(geno, got)
        plan.check()
        for name, v in _bits(want).items():
            assert torch.equal(v, _bits(got[0])[name]), f"{name}: {width} columns"
        del plan
        arena.close()


def test_segments_under_capture(tgw):
    n, m, p = 70_001, 4096, 8
    g = torch.Generator(device="cuda").manual_seed(2)
    geno = torch.randint(0, 256, (m, (n + 63) // 64 * 16), generator=g, device="cuda", dtype=torch.uint8)
    cov = tgw.fit_covariates(torch.randn((5, n), generator=g, device="cuda", dtype=torch.float64).t())
    panel = tgw.prepare_phenotypes(cov, torch.randn((p, n), generator=g, device="cuda").t(), "split8")
    plan = tgw.Plan([panel])
    want = tgw.scan(plan, geno)[0]
    outs = tgw.make_outputs([p], m)
    plan.scan(geno, outs)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        plan.scan(geno, outs)
    for _ in range(3):
        for v in outs[0].values():
            v.fill_(7.0)
        graph.replay()
        torch.cuda.synchronize()
        for name, v in _bits(want).items():
            assert torch.equal(v, _bits(outs[0])[name]), name
        plan.check()
