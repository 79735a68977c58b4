"""The error of the first iterate must not depend on the tiles that the
tridiagonal reduction takes: 64 matrices of order 512 share a launch with
256-row tiles (192 in double), one alone has 64-row tiles.

The matrix is rounded once per 32 columns in small tiles and once per 8 in
large ones.  Against the other errors of the factor (v, w, the products, the
eigenvectors) even one rounding per column is no more than half of the total,
so with an eighth of those roundings' variance the error may grow by 6 %; with
one per column it grows by a third."""

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_first_iterate_in_a_batch(prec):
    import torch
    import paper_2607_12430_amd as msq
    b, n = 64, 512
    g = torch.Generator(device="cuda")
    g.manual_seed(77)
    lam = torch.logspace(-2, 2, n, device="cuda", dtype=torch.float64)
    a, root = [], []
    for _ in range(b):
        q, _ = torch.linalg.qr(torch.randn(n, n, generator=g, device="cuda", dtype=torch.float64))
        qt = q.T.contiguous()
        m = (q * lam) @ qt
        a.append(0.5 * (m + m.T))
        root.append((q * lam.sqrt()) @ qt)

    def first(x):
        return msq.sqrtm(x.contiguous(), prec=prec, structure="hpd", maxit=0, tol=-1.0, fallback=False,
                         allow_fail=True)[0]

    def err(x, r):
        return float(torch.linalg.matrix_norm(x - r) / torch.linalg.matrix_norm(r))

    print(f"[tridiag error] {prec} {b} x {n}", flush=True)
    together = first(torch.stack(a))
    eb = sum(err(together[i], root[i]) for i in range(b)) / b
    es = sum(err(first(a[i]), root[i]) for i in range(b)) / b
    print(f"[tridiag error] batch {eb:.3e} alone {es:.3e}", flush=True)
    assert eb <= 1.12 * es
