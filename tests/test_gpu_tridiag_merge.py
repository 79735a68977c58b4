"""The tridiagonal eigensolver where its recursion changes shape: a leaf next to
a merge of one row more, halves that end inside a tile of the merge products,
merges that rotate columns next to merges that do not, entries whose scale
leaves the range of a squared double."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _check(msq, d, e, prec):
    n = d.size
    print(f"[tridiag merge] {prec} n={n}", flush=True)
    lam, z = msq.test_stedc(d, e, prec)
    if prec == "fp32":
        d, e = d.astype(np.float32).astype(np.float64), e.astype(np.float32).astype(np.float64)
    t = np.diag(d) + np.diag(e, 1) + np.diag(e, -1)
    u = 6e-8 if prec == "fp32" else 1.1e-16
    nt = np.abs(t).max()
    ref = nt * np.linalg.eigvalsh(t / nt)
    z = z.astype(np.float64)
    # the couplings of a merge are rows of Z, kept in the working precision
    assert np.abs(lam - ref).max() <= (50 * n * 1.1e-16 + (20 * n * u if prec == "fp32" else 0)) * 3 * nt
    assert np.linalg.norm(z.T @ z - np.eye(n)) <= 50 * n * u
    assert np.linalg.norm(t / nt @ z - z * (lam / nt)) <= 150 * n * u


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("n", [16, 17, 34, 64, 66, 127, 191, 260, 517])
def test_sizes(prec, n):
    import paper_2607_12430_amd as msq
    r = np.random.default_rng(n)
    _check(msq, r.standard_normal(n), r.standard_normal(n - 1), prec)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_rotations_in_some_merges(prec):
    import paper_2607_12430_amd as msq
    r = np.random.default_rng(5)
    # equal diagonals and couplings in the first half only
    d = np.concatenate([np.full(130, 2.0), r.standard_normal(131)])
    e = np.concatenate([np.full(130, 1.0), r.standard_normal(130)])
    _check(msq, d, e, prec)


@pytest.mark.parametrize("scale", [1e-200, 1e200])
def test_scale(scale):
    import paper_2607_12430_amd as msq
    r = np.random.default_rng(7)
    _check(msq, scale * r.standard_normal(32), scale * r.standard_normal(31), "fp64")


def test_underflowing_rotation():
    import paper_2607_12430_amd as msq
    # zero diagonal with couplings far below the largest one
    e = 10.0 ** -np.linspace(0, 300, 23)
    _check(msq, np.zeros(24), e, "fp64")
