"""The FP64 path of covariate-collinear markers at the edges of its work items
(16 listed markers x 64 columns, 16 ranges of sample chunks, 16-slot tiles of
the covariate basis), against the FP64 oracle at the default tolerances."""
import numpy as np
import pytest

from synth import pack_codes_np, row_bytes_for
from tests.gpu_common import compare, decode_codes, gpu_scan, lib, oracle_scan, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tgw():
    t = lib()
    t.init()
    return t


@pytest.mark.parametrize("n,p,k,listed,precision", [
    (130, 1, 1, 1, "split8"),       # three chunks (idle ranges), one marker, one column
    (700, 63, 2, 15, "split"),      # a group and a column item not quite full
    (1024, 64, 3, 16, "split16"),   # exactly full, no ragged chunk
    (1030, 65, 15, 17, "split8"),   # one more of each; q = 16: one full slot tile
    (1500, 33, 16, 33, "fp32"),     # q = 17: two slot tiles; columns end in the item's first block
    (1111, 129, 31, 40, "split8"),  # q = 32: every slot
])
def test_redo_item_edges(tgw, n, p, k, listed, precision):
    say(f"case: FP64 path n={n} p={p} k={k} listed={listed} {precision}")
    rng = np.random.default_rng(n + p)
    m = listed + 20
    maf = rng.uniform(0.1, 0.5, m)
    codes = rng.binomial(2, maf[:, None], size=(m, n)).astype(np.uint8)
    codes[0] = rng.binomial(2, 0.4, size=n)
    # markers 1 .. listed - 1 follow marker 0: each sample keeps its call with probability 0.75 to 0.95
    for i in range(1, listed):
        keep = rng.random(n) < rng.uniform(0.75, 0.95)
        codes[i] = np.where(keep, codes[0], codes[i])
    codes[rng.random((m, n)) < 0.01] = 3
    lead = decode_codes(codes[0])
    C = rng.standard_normal((n, k))
    C[:, 0] = np.where(np.isnan(lead), np.nanmean(lead), lead) + 0.05 * rng.standard_normal(n)
    Y = (rng.standard_normal((n, p)) + 0.3 * C[:, :1]).astype(np.float32)
    ref = oracle_scan(codes, C, Y)
    ratio = ref["h"] ** 2 / ref["gc2"]
    say(f"{int((ratio < 0.5).sum())} of {m} markers below one half")
    assert (ratio[:listed] < 0.55).all() and (ratio[:listed] < 0.5).sum() >= max(1, listed - 3)
    res, _, _ = gpu_scan(C, [Y], pack_codes_np(codes, row_bytes_for(n)), precision)
    compare(res[0], ref, ref["df"], f"redo n={n} p={p} k={k} ")
