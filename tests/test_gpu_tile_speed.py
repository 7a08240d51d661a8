"""The automatic choice of tiles against the plan's default tile: it may not be
the slower one.  Both are timed in turn; 15 % are allowed for the clock and for
what the choice's cost estimate does not see."""
import statistics

import pytest
import torch

from tests.gpu_common import lib, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tgw():
    t = lib()
    t.init()
    return t


def _ratio(tgw, precision, code, n, m, p, topk):
    """Time of the automatic choice over the default tile's."""
    g = torch.Generator(device="cuda").manual_seed(n + m + p)
    row = (n + 63) // 64 * (64 if code == "dosage8" else 16)
    c = tgw.CODE_DOSAGE8 if code == "dosage8" else tgw.CODE_DOSAGE
    geno = torch.randint(0, 256, (m, row), generator=g, device="cuda", dtype=torch.uint8)
    cov = tgw.fit_covariates(torch.randn((10, n), generator=g, device="cuda", dtype=torch.float64).t())
    panel = tgw.prepare_phenotypes(cov, torch.randn((p, n), generator=g, device="cuda").t(), precision)
    plans = [tgw.Plan([panel]), tgw.Plan([panel], tile=2 if code == "dosage8" else 0)]
    outs = [{"topk": w} for w in tgw.make_topk([p], topk)] if topk else tgw.make_outputs([p], m)

    def time_of(plan, reps):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(reps):
            if topk:
                outs[0]["topk"].zero_()
            plan.scan(geno, outs, code=c)
        b.record()
        b.synchronize()
        return a.elapsed_time(b) / reps

    for plan in plans:
        time_of(plan, 2)
    reps = max(2, min(50, int(5.0 / time_of(plans[1], 2))))
    times = [[time_of(plan, reps) for plan in plans] for _ in range(7)]
    auto, named = (statistics.median(t[i] for t in times) for i in (0, 1))
    say(f"case: {precision} {code} n={n} m={m} p={p} topk={topk}: path {plans[0].debug_path(m, c, topk)}, "
        f"{auto * 1e3:.0f} us, default tile {named * 1e3:.0f} us")
    return auto / named


@pytest.mark.parametrize("precision,code,n,m,p", [
    ("split8", "dosage", 70_001, 10_000, 600),   # 70 chunks after a segment of 1,024
    ("split16", "dosage", 66_000, 10_000, 600),
    ("split8", "dosage", 131_200, 10_000, 600),  # a third segment of 2 chunks
])
def test_uneven_segments(tgw, precision, code, n, m, p):
    assert _ratio(tgw, precision, code, n, m, p, 0) < 1.15


def test_segments_over_two_launches(tgw):
    """On 256 x 64 tiles the buffer for the segments' sums holds 512 of the 544
    tiles, and the rest would take a whole round of their own."""
    assert _ratio(tgw, "split8", "dosage", 80_000, 2000, 4300, 0) < 1.15


@pytest.mark.parametrize("precision,code,n,m,p,topk", [
    ("split8", "dosage", 500, 30_000, 1, 50),     # many waves at one list
    ("split", "dosage", 500, 30_000, 20, 10),
    ("split16", "dosage", 500, 100_000, 40, 50),
    ("fp32", "dosage", 1000, 2000, 20_480, 10),   # short sums, long lists
    ("split8", "dosage", 8000, 500, 20_480, 10),
    ("split8", "dosage", 48_190, 985, 8419, 1),   # half a round of wide tiles, long sums
    ("split16", "dosage8", 1500, 2000, 5000, 50),
    ("split16", "dosage8", 1000, 1301, 18_643, 10),
    ("split8", "dosage8", 500, 60_000, 300, 10),
    ("split8", "dosage", 60_000, 10_000, 1000, 0),  # a full round of wide tiles, long sums
    ("fp32", "dosage8", 1000, 3000, 2000, 0),
])
def test_outputs_and_lengths(tgw, precision, code, n, m, p, topk):
    assert _ratio(tgw, precision, code, n, m, p, topk) < 1.15


@pytest.mark.parametrize("precision,code,n,m,p,topk", [
    ("split16", "dosage", 1000, 8000, 7000, 50),
    ("split8", "dosage8", 2000, 40_000, 4600, 50),
    ("fp32", "dosage", 1000, 1500, 8000, 10),
    ("fp32", "dosage8", 2000, 600, 16_000, 10),
])
def test_lists_take_a_fast_shape(tgw, precision, code, n, m, p, topk):
    """Of the default tile and the five small ones, the automatic choice is the
    fastest or near it (20 %)."""
    g = torch.Generator(device="cuda").manual_seed(n + m + p)
    row = (n + 63) // 64 * (64 if code == "dosage8" else 16)
    c = tgw.CODE_DOSAGE8 if code == "dosage8" else tgw.CODE_DOSAGE
    geno = torch.randint(0, 256, (m, row), generator=g, device="cuda", dtype=torch.uint8)
    cov = tgw.fit_covariates(torch.randn((10, n), generator=g, device="cuda", dtype=torch.float64).t())
    plan = tgw.Plan([tgw.prepare_phenotypes(cov, torch.randn((p, n), generator=g, device="cuda").t(), precision)])
    words = tgw.make_topk([p], topk)[0]
    choice = plan.debug_path(m, c, topk)
    times = {}
    for path in [*range(6)] * 4:
        plan.debug_set_path(path)
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        words.zero_()
        a.record()
        plan.scan(geno, [{"topk": words}], code=c)
        b.record()
        b.synchronize()
        times.setdefault(path, []).append(a.elapsed_time(b))
    times = {path: min(t) for path, t in times.items()}
    say(f"case: {precision} {code} n={n} m={m} p={p} topk={topk}: path {choice}, ms {times}")
    assert times[choice] < 1.2 * min(times.values())
