"""A tridiagonal matrix with an Inf or NaN: the divide and conquer places columns
by comparisons, so it must not run on such values.  Its eigenvalues are NaN and
its eigenvectors orthonormal; nothing outside its arrays is touched (a finite
matrix solved next is solved right)."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("n", [1, 2, 16, 17, 33, 64, 200, 700])
@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
def test_eigensolver(prec, n, bad):
    import paper_2607_12430_amd as msq
    rng = np.random.default_rng(n)
    d, e = rng.standard_normal(n), rng.standard_normal(n - 1)
    t = np.diag(d) + np.diag(e, 1) + np.diag(e, -1)
    print(f"[tridiag nonfinite] {prec} n={n} {bad}", flush=True)
    for where in ("d0", "dn", "e"):
        d2, e2 = d.copy(), e.copy()
        if where == "e":
            if n == 1:
                continue
            e2[n // 2 - 1] = bad
        else:
            d2[0 if where == "d0" else -1] = bad
        lam, z = msq.test_stedc(d2, e2, prec)
        assert np.isnan(lam).all()
        z = z.astype(np.float64)
        assert np.abs(z.T @ z - np.eye(n)).max() <= 1e-6
    lam, _ = msq.test_stedc(d, e, prec)
    u = 2.0 ** -24 if prec == "fp32" else 2.0 ** -53
    assert np.abs(lam - np.linalg.eigvalsh(t)).max() <= 4 * n * u * np.abs(t).sum(axis=0).max() + 1e-12
