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
