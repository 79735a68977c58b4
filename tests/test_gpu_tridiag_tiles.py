"""The tridiagonal reduction where its launch shape changes: register tails of
64, 128, 192 and 256 rows (192 in double), tiles that do not divide the
order, changes of the tile size on the way down, batches in several launches."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("n", [2, 3, 63, 64, 65, 128, 129, 192, 193, 256, 257, 270, 385, 640, 1000])
def test_spectrum(prec, n):
    import paper_2607_12430_amd as msq
    rng = np.random.default_rng(n)
    a = rng.standard_normal((n, n))
    a = a + a.T
    if prec == "fp32":
        a = a.astype(np.float32).astype(np.float64)
    print(f"[tridiag tiles] {prec} n={n}", flush=True)
    d, e, _ = msq.test_sytrd(a, prec=prec)
    t = np.diag(d.astype(np.float64)) + np.diag(e.astype(np.float64), 1) + np.diag(e.astype(np.float64), -1)
    lam = np.linalg.eigvalsh(a)
    u = 2.0 ** -24 if prec == "fp32" else 2.0 ** -53
    # backward error of a Householder reduction: a modest multiple of n u
    assert np.max(np.abs(np.linalg.eigvalsh(t) - lam)) <= 2 * n * u * np.max(np.abs(lam))


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_largest_order(prec):
    import torch
    import paper_2607_12430_amd as msq
    n = 4225
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    b = torch.randn(n, n, generator=g, device="cuda", dtype=torch.float64) / n ** 0.5
    a = (b @ b.T.contiguous() + torch.eye(n, device="cuda", dtype=torch.float64))
    a = (0.5 * (a + a.T)).contiguous()
    _, info = msq.sqrtm(a, prec=prec, structure="hpd", fallback=False)
    assert info["status"] == "ok" and info["relres"] <= 1e-13


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("b,n", [(3, 257), (30, 500), (70, 290)])
def test_batch(prec, b, n):
    import torch
    import paper_2607_12430_amd as msq
    g = torch.Generator(device="cuda")
    g.manual_seed(b)
    z = torch.randn(b, n, n, generator=g, device="cuda", dtype=torch.float64) / n ** 0.5
    a = torch.stack([m @ m.T.contiguous() for m in z]) + torch.eye(n, device="cuda", dtype=torch.float64)
    a = (0.5 * (a + a.mT)).contiguous()
    print(f"[tridiag tiles] batch {prec} {b} x {n}", flush=True)
    x, info = msq.sqrtm(a, prec=prec, structure="hpd", fallback=False)
    assert info["status"] == "ok" and info["relres"] <= 1e-13
    for k in (0, b // 2, b - 1):
        r = torch.linalg.matrix_norm(x[k] @ x[k] - a[k]) / torch.linalg.matrix_norm(a[k])
        assert float(r) <= 1e-13
