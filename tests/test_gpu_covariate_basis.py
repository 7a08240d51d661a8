"""The covariate basis Q at the edges of its tiles and of its two
factorizations (Cholesky twice; Householder for ill-conditioned covariates),
against numpy's Householder QR, column signs included."""
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


def _case(kind, n, k):
    rng = np.random.default_rng(n + k)
    C = rng.standard_normal((n, k))
    if kind == "scaled":       # units far apart, offsets, correlated pairs
        C *= 10.0 ** rng.uniform(-4, 4, k)
        C[:, 0] += 20.0 * C[:, 0].std()
        C[:, -1] = C[:, 0] + C[:, 0].std() * 0.05 * rng.standard_normal(n)
    if kind == "collinear":    # condition about 1e7: the Householder QR
        C[:, -1] = C[:, 0] + 1e-7 * rng.standard_normal(n)
    if kind == "offset":       # one covariate nearly constant
        C[:, 0] = 1.0 + 1e-6 * C[:, 0]
    return C


@pytest.mark.parametrize("kind,n,k", [
    ("plain", 64, 0), ("plain", 5, 2), ("plain", 34, 31), ("plain", 65, 15), ("plain", 1000, 16),
    ("plain", 23000, 10), ("scaled", 4097, 20), ("scaled", 700, 7), ("scaled", 23001, 31),
    ("collinear", 3000, 9), ("offset", 2049, 17),
])
def test_basis_equals_householder(tgw, kind, n, k):
    say(f"case: covariate basis {kind} n={n} k={k}")
    C = _case(kind, n, k)
    X = np.concatenate([np.ones((n, 1)), C], axis=1)
    # wider than FP64 is not at hand: compare to what cond(X) rounding errors of unit columns allow
    unit = X / np.linalg.norm(X, axis=0)
    cond = np.linalg.cond(unit)
    want = np.linalg.qr(X)[0]  # R_jj = -sign(pivot) |R_jj|
    Cd = torch.from_numpy(C).cuda() if k else None
    cov = tgw.fit_covariates(Cd, n_samples=n)
    Q = cov.Q().cpu().numpy()
    ortho = np.abs(Q.T @ Q - np.eye(k + 1)).max()
    span = np.abs(unit - Q @ (Q.T @ unit)).max()
    diff = np.abs(Q - want).max()
    say(f"cond {cond:.2g}: |Q'Q - I| {ortho:.2g}, outside the span {span:.2g}, |Q - numpy| {diff:.2g}")
    assert ortho < 1e-13 * (k + 1)
    assert span < 1e-14 * (k + 1)
    assert diff < 1e-14 * (k + 1) * max(cond, 1.0)
    again = tgw.fit_covariates(Cd, n_samples=n).Q().cpu().numpy()
    np.testing.assert_array_equal(Q, again)


@pytest.mark.parametrize("kind", ["copy", "sum", "constant", "zero", "tiny"])
def test_rank_deficient_covariates(tgw, kind):
    rng = np.random.default_rng(9)
    C = rng.standard_normal((1500, 6))
    C[:, 4] = {"copy": C[:, 1], "sum": C[:, 0] - 2 * C[:, 2], "constant": np.full(1500, 3.0),
               "zero": np.zeros(1500), "tiny": 1e-12 * C[:, 4]}[kind]
    with pytest.raises(tgw.TgwError) as e:
        tgw.fit_covariates(torch.from_numpy(C).cuda())
    assert e.value.status == tgw.ERR_RANK_DEFICIENT


@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_nonfinite_covariates(tgw, value):
    C = np.random.default_rng(4).standard_normal((700, 18))
    C[699, 17] = value
    with pytest.raises(tgw.TgwError) as e:
        tgw.fit_covariates(torch.from_numpy(C).cuda())
    assert e.value.status == tgw.ERR_NONFINITE
