"""Timed cases of the association scan, over the range its users run it in.

A case is a dict of plain values:

  kind     "scan"     tgw.Plan.scan on a kept plan (panel prepared, workspace
                      and output buffers in hand), as in a loop over marker
                      blocks;
           "session"  fit_covariates + prepare_phenotypes + Plan + scan +
                      check: a new panel (or new covariates) against the
                      markers of a region;
           "bed"      tgw.scan_bed: the markers of a PLINK .bed file (page
                      cache) with a sample selection, streamed through a kept
                      plan.
  n, m, k  samples, markers, covariates (without the intercept)
  p        phenotypes; with panels > 1 the largest panel's: the others are
           log-uniform between 32 and p, their covariates uniform in 3..k
  panels   phenotype panels of the plan
  prec     precision of the contraction (tgw.prepare_phenotypes)
  code     genotype rows: "dosage" (2 bits), "plink" (2 bits, .bed order),
           "dosage8" (8-bit dosages)
  y64      phenotypes handed over in FP64 (else FP32)
  topk     0: dense r, beta, SE, t, -log10 p; else the top-k list per
           phenotype instead (panels whose dense outputs nobody keeps)
  leads    lead markers of the region that join the covariates (conditional
           analysis); half of the region's markers are then in linkage
           disequilibrium with one of them

Inputs: minor allele frequencies U(0.05, 0.5), 1 % missing calls, phenotypes
from 20 causal markers, the covariates and noise; large panels have a shared
factor in half of their columns.  All handles take their device memory from
one arena over a torch tensor that the process keeps, as bench.py does.
"""
import math
import os
import random
import tempfile

import numpy as np
import torch

from paper_2604_21095_amd import tgw

_NAMES = ("r", "beta", "se", "t", "nlog10p")
_CODES = {"dosage": tgw.CODE_DOSAGE, "plink": tgw.CODE_PLINK_BED, "dosage8": tgw.CODE_DOSAGE8}
_PLINK = (0, 2, 3, 1)  # .bed code of 0, 1, 2 copies and of a missing call
_ARENA_GIB = 32
_arena = None


def _case(name, kind="scan", n=23000, m=4096, k=10, p=1, panels=1, prec="split8", code="dosage", y64=False, topk=0,
          leads=0):
    c = {"kind": kind, "n": n, "m": m, "k": k, "p": p, "panels": panels, "prec": prec, "code": code, "y64": y64,
         "topk": topk, "leads": leads}
    return {"name": name, **c} if name else c


def listed():
    return [
        # a small study in full, in the binding's default precision: the smallest call, where launches count
        _case("small study", n=2000, m=5000, p=16, k=4, prec="split"),
        # the ordinary genome-wide scan of one trait, PLINK-coded rows
        _case("one trait", m=100_000, p=1, code="plink"),
        # a handful of traits with more covariates, a ragged panel width
        _case("small panel", m=65_536, p=45, k=20),
        # a biobank-sized cohort (odd sample count), a few traits
        _case("biobank", n=500_001, m=4096, p=8, k=20),
        # the plain FP32 form on a medium panel
        _case("fp32 panel", m=16_384, p=500, prec="fp32"),
        # the imaging panel of the benchmark cohort, dense outputs: a large block of markers
        _case("imaging panel", m=100_000, p=2048),
        # the full imaging panel at its width, of which only the top tests are kept
        _case("panel scale", m=16_384, p=20_480, topk=10),
        # many uneven panels with covariates of their own in one launch sequence
        _case("batch of panels", m=10_000, p=2048, panels=12, k=20),
        # imputed dosages, one byte per sample, in the FP16 split
        _case("dosages", m=20_000, p=256, prec="split16", code="dosage8"),
        # a .bed file with a sample selection, streamed
        _case("bed stream", "bed", m=24_000, p=128),
        # a new phenotype panel (FP64 as most tables arrive) against a candidate region
        _case("new panel", "session", m=2000, p=2048, y64=True),
        # conditional analysis: lead markers join the covariates, the region around them is scanned again
        _case("conditional", "session", m=3000, p=300, k=10, leads=3),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the same ranges; its operations, inputs and outputs stay within the listed ones'."""
    kind = rng.choice(["scan"] * 7 + ["session"] * 2 + ["bed"])
    while True:
        prec = rng.choice(["split8", "split8", "split", "split16", "fp32"])
        code = rng.choice(["dosage", "plink", "dosage8"] if prec != "split" else ["dosage", "plink"])
        panels, topk, leads, y64 = 1, 0, 0, rng.random() < 0.25
        n = _log_uniform(rng, 1000, 500_001) if kind == "scan" else _log_uniform(rng, 1000, 40_000)
        m = _log_uniform(rng, 500, 100_000)
        p = _log_uniform(rng, 1, 20_480)
        k = rng.randint(0, 20)
        if kind == "scan":
            if p >= 4096:
                topk = rng.choice([1, 10, 50])
            elif p >= 64 and k >= 3 and rng.random() < 0.4:
                panels = rng.randint(2, 12)
        elif kind == "session":
            m, p = _log_uniform(rng, 200, 6000), _log_uniform(rng, 1, 4096)
            leads = rng.choice([0, 0, 1, 4])
            if leads:
                m, p = min(m, 69_000_000 // n), min(p, 300)
        else:
            m, p, code = _log_uniform(rng, 2000, 24_000), _log_uniform(rng, 1, 1024), "plink"
        c = _case("", kind, n, m, k, p, panels, prec, code, y64, topk, leads)
        tests = m * sum(_panel_sizes(c))
        slow = {"fp32": 7.0, "split": 1.4, "split16": 1.4, "split8": 1.0}[prec]
        rows = m * n * (1.0 if code == "dosage8" else 0.25)
        if slow * tests * n <= 3.5e12 and (topk or tests <= 2.0e8) and rows <= 6e8:
            return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _panel_sizes(c):
    rng = random.Random("%d/%d" % (c["panels"], c["p"]))
    return [c["p"]] + [_log_uniform(rng, 32, max(32, c["p"])) for _ in range(c["panels"] - 1)]


def _panel_covariates(c):
    rng = random.Random("%d/%d/%d" % (c["panels"], c["p"], c["k"]))
    return [c["k"]] + [rng.randint(3, max(3, c["k"])) for _ in range(c["panels"] - 1)]


def _generator(*key):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(np.random.SeedSequence([int(x) for x in key]).generate_state(1, np.uint32)[0]))
    return g


def _chunks(m, n):
    step = max(1, min(m, 60_000_000 // n))
    return [(a, min(m, a + step)) for a in range(0, m, step)]


def _draw_calls(rows, n, g):
    """(rows, n) copies of the counted allele, 3 = missing."""
    maf = 0.05 + 0.45 * torch.rand((rows, 1), device="cuda", generator=g)
    calls = (torch.rand((rows, n), device="cuda", generator=g) < maf).to(torch.uint8)
    calls += torch.rand((rows, n), device="cuda", generator=g) < maf
    calls[torch.rand((rows, n), device="cuda", generator=g) < 0.01] = 3
    return calls


def _pack(c, calls, row_bytes, g):
    """Rows in the case's code; bytes past the last sample hold missing calls."""
    rows, n = calls.shape
    if c["code"] == "dosage8":
        out = torch.full((rows, row_bytes), 255, dtype=torch.uint8, device="cuda")
        q = calls.to(torch.int16) * 127 + torch.randint(-24, 25, calls.shape, device="cuda", generator=g,
                                                        dtype=torch.int16)
        out[:, :n] = torch.where(calls == 3, 255, q.clamp(0, 254)).to(torch.uint8)
        return out
    missing = 1 if c["code"] == "plink" else 3
    codes = torch.full((rows, row_bytes * 4), missing, dtype=torch.uint8, device="cuda")
    if c["code"] == "plink":
        calls = torch.tensor(_PLINK, dtype=torch.uint8, device="cuda")[calls.long()]
    codes[:, :n] = calls
    codes = codes.view(rows, row_bytes, 4)
    return codes[..., 0] | codes[..., 1] << 2 | codes[..., 2] << 4 | codes[..., 3] << 6


def _row_bytes(c, n):
    return (n + 63) // 64 * (64 if c["code"] == "dosage8" else 16)


def _calls_of(c, rows, n):
    """FP64 (rows, n) genotypes of packed rows, NaN = missing."""
    if c["code"] == "dosage8":
        q = rows[:, :n].double()
        return torch.where(q == 255, torch.nan, q / 127.0)
    codes = torch.stack([rows >> s & 3 for s in (0, 2, 4, 6)], dim=-1).flatten(1)[:, :n]
    values = (0.0, math.nan, 1.0, 2.0) if c["code"] == "plink" else (0.0, 1.0, 2.0, math.nan)
    return torch.tensor(values, dtype=torch.float64, device="cuda")[codes.long()]


def _imputed(g):
    mean = torch.nanmean(g, dim=1, keepdim=True)
    return torch.where(torch.isnan(g), mean, g)


def _draw_geno(c, seed, n):
    g = _generator(seed, 1)
    leads = _draw_calls(c["leads"], n, g) if c["leads"] else None
    geno = torch.empty((c["m"], _row_bytes(c, n)), dtype=torch.uint8, device="cuda")
    for a, b in _chunks(c["m"], n):
        calls = _draw_calls(b - a, n, g)
        if leads is not None:  # every second marker follows a lead: each sample keeps the lead's call or its own draw
            rows = torch.arange(a, b, device="cuda")
            keep = torch.where(rows % 2 == 0, 0.3 + 0.68 * torch.rand(b - a, device="cuda", generator=g), 0.0)
            own = torch.rand((b - a, n), device="cuda", generator=g) >= keep[:, None]
            calls = torch.where(own, calls, leads[rows // 2 % c["leads"]])
            for j in range(c["leads"]):  # the leads themselves are markers of the region
                at = (2 * j + 1) * c["m"] // (2 * c["leads"])
                if a <= at < b:
                    calls[at - a] = leads[j]
        geno[a:b] = _pack(c, calls, geno.shape[1], g)
    return geno


def _draw_panel(c, seed, j, n, geno):
    """Covariates (n, k) FP64 and phenotypes (n, p) of panel j, samples of a column contiguous."""
    g = _generator(seed, 2, j)
    k, p = _panel_covariates(c)[j], _panel_sizes(c)[j]
    cov = torch.randn((k, n), device="cuda", generator=g, dtype=torch.float64)
    y = torch.randn((p, n), device="cuda", generator=g)
    at = torch.arange(20, device="cuda") * (c["m"] - 1) // 19
    causal = _imputed(_calls_of(c, geno[at], n)).float()
    effects = math.sqrt(0.05) * torch.randn((p, 20), device="cuda", generator=g)
    y += effects @ (causal - causal.mean(dim=1, keepdim=True))
    if k:
        y += torch.randn((p, k), device="cuda", generator=g) @ cov.float()
    if p >= 4096:
        y[: p // 2] += torch.randn((p // 2, 64), device="cuda", generator=g) @ (
            torch.randn((64, n), device="cuda", generator=g) / 8.0)
    if c["leads"]:
        at = torch.tensor([(2 * i + 1) * c["m"] // (2 * c["leads"]) for i in range(c["leads"])], device="cuda")
        cov = torch.cat([cov, _imputed(_calls_of(c, geno[at], n))])
    return (cov.t() if cov.shape[0] else None), (y.double() if c["y64"] else y).t()


def _file_samples(c, seed):
    """Samples of the .bed file and the file sample of each scan sample: about a tenth of the file is left out."""
    n_file = c["n"] + c["n"] // 9
    keep = np.sort(np.random.default_rng([int(seed), 3]).permutation(n_file)[: c["n"]])
    return n_file, keep


def _inputs(c, seed):
    """(geno, [(C, Y) per panel]) of the samples that are scanned."""
    geno = _draw_geno(c, seed, c["n"])
    return geno, [_draw_panel(c, seed, j, c["n"], geno) for j in range(c["panels"])]


def _write_bed(c, seed, geno):
    """The scanned samples' calls in a .bed file among samples that the scan leaves out; an open handle."""
    n_file, keep = _file_samples(c, seed)
    at = torch.from_numpy(keep).cuda()
    shifts = torch.tensor([0, 2, 4, 6], device="cuda", dtype=torch.uint8)
    fd, path = tempfile.mkstemp(suffix=".bed")
    with os.fdopen(fd, "wb") as f:
        f.write(bytes([0x6C, 0x1B, 0x01]))
        for a, b in _chunks(c["m"], n_file):
            codes = torch.zeros((b - a, (n_file + 3) // 4 * 4), dtype=torch.uint8, device="cuda")
            codes[:, at] = (geno[a:b, :, None] >> shifts & 3).flatten(1)[:, : c["n"]]
            q = codes.view(b - a, -1, 4)
            f.write((q[..., 0] | q[..., 1] << 2 | q[..., 2] << 4 | q[..., 3] << 6).cpu().numpy().tobytes())
    bed = tgw.Bed(path, n_file)
    os.unlink(path)  # the handle keeps the file open
    bed.select(keep.tolist())
    return bed


def _with_code(c):
    return {**c, "code": "plink"} if c["kind"] == "bed" else c


# ---------------------------------------------------------------------------
# the timed passes
# ---------------------------------------------------------------------------
def prepare(case, seed):
    global _arena
    c = _with_code(case)
    if _arena is None:
        tgw.init()
        _arena = tgw.torch_arena(_ARENA_GIB << 30).register()
    geno, panels = _inputs(c, seed)
    state = {"case": c, "geno": geno, "code": _CODES[c["code"]]}
    if c["kind"] == "session":
        state["C"], state["Y"] = panels[0]
        return state
    handles = []
    for C, Y in panels:
        handles.append(tgw.prepare_phenotypes(tgw.fit_covariates(C, n_samples=c["n"]), Y, c["prec"]))
    del panels, C, Y
    state["plan"] = tgw.Plan(handles)
    if c["topk"]:
        state["outs"] = [{"topk": w} for w in tgw.make_topk([h.n_pheno for h in handles], c["topk"])]
    else:
        state["outs"] = tgw.make_outputs([h.n_pheno for h in handles], c["m"])
    if c["kind"] == "bed":
        state["bed"] = _write_bed(c, seed, geno)
        del state["geno"]
    return state


def run(state):
    c = state["case"]
    if c["kind"] == "session":
        cov = tgw.fit_covariates(state["C"], n_samples=c["n"])
        plan = tgw.Plan([tgw.prepare_phenotypes(cov, state["Y"], c["prec"])])
        outs = tgw.scan(plan, state["geno"], code=state["code"])
        plan.check()
        return {"Q": cov.Q(), **outs[0]}
    plan, outs = state["plan"], state["outs"]
    if c["topk"]:
        outs[0]["topk"].zero_()
    if c["kind"] == "bed":
        tgw.scan_bed(plan, state["bed"], outs, block_markers=4096, n_threads=8)
    else:
        plan.scan(state["geno"], outs, code=state["code"])
    if c["topk"]:
        # the lists' values: tests of one phenotype that tie within rounding may trade places, and with them their markers
        return {"nlog10p": tgw.read_topk(plan.panels[0], outs[0]["topk"])[0]}
    return outs if len(outs) > 1 else outs[0]


def work(case):
    c = _with_code(case)
    sizes = _panel_sizes(c)
    n, m, p = c["n"], c["m"], sum(sizes)
    n_rows = _file_samples(c, 0)[0] if c["kind"] == "bed" else n
    read = m * n_rows * (1.0 if c["code"] == "dosage8" else 0.25)
    written = 12.0 * p * c["topk"] if c["topk"] else 20.0 * m * p
    flops = 2.0 * n * m * p
    if c["kind"] == "session":
        q = c["k"] + c["leads"] + 1
        read += n * p * (8.0 if c["y64"] else 4.0) + 8.0 * n * (q - 1)
        written += 8.0 * n * q
        flops += 4.0 * n * q * (p + q)
    else:
        read += n * p * (3.0 if c["prec"] == "split8" else 4.0)
    return {"bytes": read + written, "flops": flops}


# ---------------------------------------------------------------------------
# the same values in 64 bits
# ---------------------------------------------------------------------------
def _beta_fraction(x, a, b):
    """Continued fraction of the incomplete beta function (DLMF 8.17.22), by the modified Lentz method."""
    tiny = 1e-300
    c = torch.ones_like(x)
    d = 1.0 - (a + b) * x / (a + 1.0)
    d = 1.0 / torch.where(d.abs() < tiny, tiny, d)
    h = d.clone()
    for i in range(1, 4000):
        for num in (i * (b - i) * x / ((a + 2 * i - 1) * (a + 2 * i)),
                    -(a + i) * (a + b + i) * x / ((a + 2 * i) * (a + 2 * i + 1))):
            d = 1.0 + num * d
            d = 1.0 / torch.where(d.abs() < tiny, tiny, d)
            c = 1.0 + num / c
            c = torch.where(c.abs() < tiny, tiny, c)
            h = h * d * c
        if float((d * c - 1.0).abs().max()) < 1e-15:
            break
    return h


def _nlog10p(t, df):
    """-log10 of the two-sided Student-t p-value: I_x(df/2, 1/2) at x = df / (df + t^2)."""
    a, b = 0.5 * df, 0.5
    t = t.double().abs()
    t2 = t * t
    x, y = df / (df + t2), t2 / (df + t2)
    ln_front = math.lgamma(a + b) - math.lgamma(a) - math.lgamma(b) + a * -torch.log1p(t2 / df) + b * torch.log(
        y.clamp_min(1e-300))
    tail = x < (a + 1.0) / (a + b + 2.0)
    upper = ln_front + torch.log(_beta_fraction(torch.where(tail, x, 0.0), a, b) / a)
    body = torch.log1p(-torch.exp(ln_front) * _beta_fraction(torch.where(tail, 0.0, y), b, a) / b)
    return -torch.where(tail, upper, body) / math.log(10.0)


class _PValues:
    """_nlog10p over many tests at one df: cubic Hermite through 64-bit nodes below |t| = 45, in full above."""

    def __init__(self, df):
        self.df, self.h = df, 1.0 / 1024.0
        t = torch.arange(45 * 1024 + 2, device="cuda", dtype=torch.float64) * self.h
        f = _nlog10p(t, df)
        ln_pdf = math.lgamma(0.5 * (df + 1)) - math.lgamma(0.5 * df) - 0.5 * math.log(
            df * math.pi) - 0.5 * (df + 1) * torch.log1p(t * t / df)
        slope = 2.0 * torch.exp(ln_pdf + f * math.log(10.0)) / math.log(10.0) * self.h
        self.nodes = torch.stack([f, slope], dim=1)

    def __call__(self, t):
        at = t.abs()
        u = at.clamp_max(45.0).nan_to_num(0.0) / self.h
        i = u.long()
        s = u - i
        (f0, d0), (f1, d1) = self.nodes[i].unbind(-1), self.nodes[i + 1].unbind(-1)
        out = f0 + s * (d0 + s * (3 * (f1 - f0) - 2 * d0 - d1 + s * (2 * (f0 - f1) + d0 + d1)))
        far = at > 45.0
        if bool(far.any()):
            out[far] = _nlog10p(at[far], self.df)
        return torch.where(torch.isnan(at), torch.nan, out)


def _householder(C, n):
    """Q of [1 | C] with the column signs of a Householder QR (R_jj = -sign(pivot) norm)."""
    X = torch.ones((n, 1), dtype=torch.float64, device="cuda")
    return torch.linalg.qr(X if C is None else torch.cat([X, C], dim=1))[0]


def _exact_panel(c, C, Y, geno, emit):
    """emit(first row, {statistic: (rows, p)}) for blocks of markers, in 64 bits."""
    n, m = c["n"], c["m"]
    Q = _householder(C, n)
    df = n - Q.shape[1] - 1
    pv = _PValues(df)
    Y = Y.double()
    Y = Y - Y.mean(dim=0)
    Y = Y - Q @ (Q.t() @ Y)
    Y = Y - Q @ (Q.t() @ Y)
    s = Y.norm(dim=0)
    step = max(1, min(200_000_000 // n, 60_000_000 // Y.shape[1], m))
    for a in range(0, m, step):
        g = _imputed(_calls_of(c, geno[a:a + step], n))
        gc = g - g.mean(dim=1, keepdim=True)
        res = gc - (gc @ Q) @ Q.t()
        res = res - (res @ Q) @ Q.t()
        norm2 = res.square().sum(dim=1, keepdim=True)
        norm = torch.where(norm2 <= 1e-8 * gc.square().sum(dim=1, keepdim=True), torch.nan, norm2).sqrt()
        r = (res @ Y) / (norm * s)
        t = r * torch.sqrt(df / (1.0 - r * r))
        se = s * torch.sqrt((1.0 - r * r) / df) / norm
        emit(a, {"r": r, "beta": t * se, "se": se, "t": t, "nlog10p": pv(t)})
    return Q


def exact(case, seed):
    c = _with_code(case)
    geno, panels = _inputs(c, seed)
    if c["topk"]:
        best = []

        def top(a, v):
            best.append(v["nlog10p"].t().topk(min(c["topk"], v["t"].shape[0]), dim=1)[0])
            if len(best) > 1:
                best[:] = [torch.cat(best, dim=1).topk(min(c["topk"], best[0].shape[1] + best[1].shape[1]), dim=1)[0]]

        _exact_panel(c, *panels[0], geno, top)
        return {"nlog10p": best[0]}
    outs = []
    for C, Y in panels:
        o = {k: torch.empty((c["m"], Y.shape[1]), dtype=torch.float64, device="cuda") for k in _NAMES}

        def dense(a, v):
            for k in _NAMES:
                o[k][a:a + v[k].shape[0]] = v[k]

        Q = _exact_panel(c, C, Y, geno, dense)
        outs.append(o)
    if c["kind"] == "session":
        return {"Q": Q, **outs[0]}
    return outs if len(outs) > 1 else outs[0]
