"""Which kernel a scan runs: a plan made for a tile runs that tile whatever the
sizes, and every tile and small tile gives a test the same bits."""
import json

import pytest
import torch

from tests.gpu_common import lib, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tgw():
    t = lib()
    t.init()
    return t


def _inputs(tgw, code, n, m, k, p, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    row = (n + 63) // 64 * (64 if code == "dosage8" else 16)
    geno = torch.randint(0, 256, (m, row), generator=g, device="cuda", dtype=torch.uint8)
    C = torch.randn((k, n), generator=g, device="cuda", dtype=torch.float64).t()
    Y = torch.randn((p, n), generator=g, device="cuda").t()
    c = {"dosage": tgw.CODE_DOSAGE, "plink": tgw.CODE_PLINK_BED, "dosage8": tgw.CODE_DOSAGE8}[code]
    return geno, tgw.fit_covariates(C), Y, c


def _scan(tgw, plan, geno, p, code):
    out = tgw.make_outputs([p], geno.shape[0])[0]
    for v in out.values():
        v.fill_(7.0)
    plan.scan(geno, [out], code=code)
    plan.check()
    return {k: v.view(torch.int32) for k, v in out.items()}


@pytest.mark.parametrize("precision,code,tiles", [
    ("split8", "dosage", (0, 1, 6)), ("split16", "plink", (0, 1, 2, 3, 4, 5)), ("split", "dosage", (0, 1, 2)),
    ("fp32", "dosage", (0, 3, 4, 5)), ("split8", "dosage8", (0, 1)), ("split16", "dosage8", (0, 1, 2, 3)),
    ("fp32", "dosage8", (0, 3)),
])
def test_named_tile_runs(tgw, precision, code, tiles):
    """Sizes at which the automatic choice takes small tiles."""
    n, m, p = 700, 1100, 40
    geno, cov, Y, c = _inputs(tgw, code, n, m, 5, p, 1)
    panel = tgw.prepare_phenotypes(cov, Y, precision)
    assert tgw.Plan([panel]).debug_path(m, c) > 0
    for t in tiles:
        say(f"case: named tile {precision} {code} tile={t}")
        plan = tgw.Plan([panel], tile=t)
        assert plan.debug_path(m, c) == 0
        r = _scan(tgw, plan, geno, p, c)["r"].view(torch.float32)
        assert torch.isfinite(r).float().mean() > 0.9 and not (r == 7.0).any()


# shape -> (markers, column blocks)
SHAPES = {0: (128, 1), 1: (256, 1), 2: (128, 2), 3: (256, 2), 4: (128, 4)}


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
def test_small_tiles_have_the_tiles_bits(tgw, precision, code, tile, n, k):
    p = 130  # more columns than the widest small tile
    geno, cov, Y, c = _inputs(tgw, code, n, 1200, k, p, n + k)
    widths = (p, 1, 32, 33, 64, 65)
    for width in widths:
        panel = tgw.prepare_phenotypes(cov, Y[:, :width], precision)
        named = tgw.Plan([panel], tile=tile)
        for m in (1, 127, 128, 129, 257, 1200):
            assert named.debug_path(m, c) == 0
            want = _scan(tgw, named, geno[:m], width, c)
            small = tgw.Plan([panel], tile=tile)
            for shape, (_, blocks) in SHAPES.items():
                fused = precision != "fp32" and width <= 32 * blocks and shape <= 2 and not (
                    shape == 1 and (k > 15 or code == "dosage8"))
                for path in (1 + shape,) + ((17 + shape,) if fused else ()):
                    if m == 1:
                        say(f"case: small tiles {precision} {code} tile={tile} n={n} k={k} p={width} path={path}")
                    small.debug_set_path(path)
                    got = _scan(tgw, small, geno[:m], width, c)
                    for name, v in got.items():
                        assert torch.equal(v, want[name]), f"{name}: path {path}, {m} markers, {width} columns"


@pytest.mark.parametrize("little_memory", [False, True])
@pytest.mark.parametrize("precision,code,tile", [
    ("split8", "dosage", 0), ("split8", "plink", 1), ("split8", "dosage", 6), ("split16", "dosage", 0),
    ("split16", "dosage", 1), ("split8", "dosage8", 0), ("split8", "dosage8", 1), ("split16", "dosage8", 0),
    ("split16", "dosage8", 1),
])
def test_segments_on_every_wide_tile(tgw, precision, code, tile, little_memory):
    """Three segments of the samples (so one in the middle) on the wide tiles,
    also with a buffer for fewer workgroups than CUs, against the small tiles."""
    n, m, p, k = 140_001, 3000, 300, 20
    say(f"case: wide segments {precision} {code} tile={tile} little_memory={little_memory}")
    geno, cov, Y, c = _inputs(tgw, code, n, m, k, p, 3)
    panel = tgw.prepare_phenotypes(cov, Y, precision)
    if little_memory:
        arena = tgw.torch_arena(6 << 20)
        arena.register()
    try:
        named = tgw.Plan([panel], tile=tile, block_markers=1024, tail_capacity=1024)
    finally:
        tgw.set_allocator()
    if little_memory:
        assert arena.info().n_failed >= 1
    assert named.debug_path(m, c) == 0
    want = _scan(tgw, named, geno, p, c)
    assert torch.isfinite(want["r"].view(torch.float32)).float().mean() > 0.9
    small = tgw.Plan([panel], tile=tile, block_markers=1024, tail_capacity=1024)
    small.debug_set_path(3)
    for name, v in _scan(tgw, small, geno, p, c).items():
        assert torch.equal(v, want[name]), name
    del named
    if little_memory:
        arena.close()


def test_cached_tile_leaves_the_choice_of_small_tiles(tgw, tmp_path, monkeypatch):
    """A tile from the autotuner's cache is the plan's tile, with small tiles where they are the faster ones; both
    take that tile's order of the FP8 steps."""
    n, m, p = 515, 900, 70
    geno, cov, Y, c = _inputs(tgw, "dosage", n, m, 4, p, 9)
    panel = tgw.prepare_phenotypes(cov, Y, "split8")
    cache = tmp_path / "tune.json"
    monkeypatch.setenv("TGW_TUNE_CACHE", str(cache))
    arch = torch.cuda.get_device_properties(0).gcnArchName
    cache.write_text(json.dumps({f"{arch}/npad576/cb3/np1/prec3": 6}))
    plan = tgw.Plan([panel])
    assert plan.info()["tile"] == 6 and plan.debug_path(m, c) > 0
    want = _scan(tgw, tgw.Plan([panel], tile=6), geno, p, c)
    for name, v in _scan(tgw, plan, geno, p, c).items():
        assert torch.equal(v, want[name]), name
