"""Calls in arenas that hold what the call keeps and its documented temporaries,
and nothing beyond."""
import pytest
import torch

from tests.gpu_common import lib, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tgw():
    t = lib()
    t.init()
    return t


def _blocks(*sizes):
    return sum((s + 255) // 256 * 256 for s in sizes)


@pytest.mark.parametrize("kind", ["plain", "collinear"])
@pytest.mark.parametrize("n,k", [(4, 1), (300, 31), (23_000, 10), (70_001, 20)])
def test_fit_asks_for_no_more_than_its_buffers(tgw, kind, n, k):
    """Q, the columns [1 | C], 33 KiB for the QR and the Q^T g operands; the
    same basis as in any other memory."""
    if kind == "collinear" and n < 100:
        pytest.skip("too few samples for a collinear pair")
    say(f"case: fit in exact memory {kind} n={n} k={k}")
    g = torch.Generator(device="cuda").manual_seed(n + k)
    C = torch.randn((k, n), generator=g, device="cuda", dtype=torch.float64)
    if kind == "collinear":
        C[-1] = C[0] + 1e-7 * C[-1]
    q, n_pad = k + 1, (n + 63) // 64 * 64
    hl = 1 if q <= 16 else 2
    need = _blocks(8 * q * n_pad, 8 * q * n_pad, 8 * q, 8 * (128 * 32 + 64), 256, n_pad * 128, hl * n_pad * 128,
                   hl * n_pad * 128)
    want = tgw.fit_covariates(C.t()).Q()
    arena = tgw.torch_arena(need)
    arena.register()
    try:
        cov = tgw.fit_covariates(C.t())
    finally:
        tgw.set_allocator()
    assert arena.info().n_failed == 0
    assert torch.equal(cov.Q(), want)
    del cov
    arena.close()


@pytest.mark.parametrize("precision,p", [("split8", 40), ("split16", 300)])
def test_long_cohort_plan_without_room_for_segments(tgw, precision, p):
    """A plan for 65,600 samples where one for 65,536 fits exactly: it scans
    all the same, in one run over the samples."""
    say(f"case: plan in exact memory {precision} p={p}")
    k, m = 5, 700

    def inputs(n):
        g = torch.Generator(device="cuda").manual_seed(3)
        geno = torch.randint(0, 256, (m, (n + 63) // 64 * 16), generator=g, device="cuda", dtype=torch.uint8)
        C = torch.randn((k, n), generator=g, device="cuda", dtype=torch.float64).t()
        Y = torch.randn((p, n), generator=g, device="cuda").t()
        return geno, tgw.prepare_phenotypes(tgw.fit_covariates(C), Y, precision)

    def plan_in(arena, panel):
        arena.register()
        try:
            return tgw.Plan([panel], block_markers=512, tail_capacity=1024)
        finally:
            tgw.set_allocator()

    big = tgw.torch_arena(256 << 20)
    short = plan_in(big, inputs(65_536)[1])
    need = big.info().peak
    del short
    big.close()
    geno, panel = inputs(65_600)
    want = tgw.scan(tgw.Plan([panel]), geno)[0]
    arena = tgw.torch_arena(need)
    plan = plan_in(arena, panel)
    assert arena.info().n_failed >= 1 and arena.info().in_use == need
    got = tgw.make_outputs([p], m)
    plan.scan(geno, got)
    plan.check()
    # both take under n / 16 FP32 steps of half an ulp, of random sign, on partial sums of under 4 sqrt(n)
    assert (got[0]["r"] - want["r"]).abs().max() < 4e-6
    assert torch.isfinite(got[0]["nlog10p"]).float().mean() > 0.9
    del plan
    arena.close()


@pytest.mark.parametrize("n,p,k", [(8000, 2000, 0), (4097, 4096, 15), (23_000, 20_480, 10)])
def test_preparation_scratch_stays_small(tgw, n, p, k):
    """Beside the panel, the preparation with up to 15 covariates takes 19 sums
    per column and sample segment (about 8,192 segments of 16 columns: 20 MB)
    and 40 per column: less than the 32 MiB from which on hipMalloc takes
    several hundred microseconds."""
    import ctypes

    say(f"case: scratch of the preparation n={n} p={p} k={k}")
    g = torch.Generator(device="cuda").manual_seed(1)
    C = torch.randn((k, n), generator=g, device="cuda", dtype=torch.float64).t() if k else None
    cov = tgw.fit_covariates(C, n_samples=n)
    Y = torch.randn((p, n), generator=g, device="cuda").t()
    counts = tgw.AllocCounts()
    alloc, free = tgw.debug_counting_allocator()
    tgw.set_allocator(alloc, free, ctypes.addressof(counts))
    try:
        panel = tgw.prepare_phenotypes(cov, Y, "split8")
        del panel
    finally:
        tgw.set_allocator()
    operand = (p + 31) // 32 * ((n + 63) // 64) * 6144
    assert counts.n_alloc == counts.n_free
    assert counts.bytes - operand < 32 << 20
