"""The Hessenberg reduction where its launch shape changes: one workgroup up to
order 128, 16 rows per workgroup above, rows of A beyond the registers, a
column too long for LDS, and rows that leave LDS too little for a full panel."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,n", [("fp32", 34), ("fp32", 127), ("fp32", 128), ("fp32", 129),
                                    ("fp32", 301), ("fp32", 1100), ("fp64", 98), ("fp64", 128),
                                    ("fp64", 129), ("fp64", 600), ("fp64", 3008), ("fp64", 8200)])
def test_complex_reduction(prec, n):
    import torch
    import paper_2607_12430_amd as msq
    rng = np.random.default_rng(n)
    a = (rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))) / np.sqrt(n)
    print(f"[hessenberg] complex {prec} n={n}", flush=True)
    h, q = msq.test_gehrd(a, prec=prec)
    u = 2.0 ** -24 if prec == "fp32" else 2.0 ** -53
    assert np.all(np.tril(h, -2) == 0)
    a, h, q = (torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (a, h, q))
    eye = torch.eye(n, dtype=a.dtype, device="cuda")
    assert float(torch.linalg.matrix_norm(q.mH.contiguous() @ q - eye)) <= 20 * n * u
    err = torch.linalg.matrix_norm(q @ h @ q.mH.contiguous() - a) / torch.linalg.matrix_norm(a)
    assert float(err) <= 20 * np.sqrt(n) * u


@pytest.mark.parametrize("prec,n", [("fp32", 3), ("fp32", 128), ("fp32", 129), ("fp32", 2100),
                                    ("fp64", 128), ("fp64", 1100)])
def test_real_reduction_through_the_schur_form(prec, n):
    import torch
    import paper_2607_12430_amd as msq
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    a = 2 * torch.eye(n, device="cuda", dtype=torch.float64)
    a = a + torch.randn(n, n, generator=g, device="cuda", dtype=torch.float64) / n ** 0.5
    print(f"[hessenberg] real {prec} n={n}", flush=True)
    f = msq.factor(a, prec=prec, structure="general")
    q, _, _ = f.export(single=prec == "fp32", structure="general")
    q = torch.from_numpy(q[0].astype(np.float64)).cuda()
    u = 2.0 ** -24 if prec == "fp32" else 2.0 ** -53
    eye = torch.eye(n, dtype=torch.float64, device="cuda")
    assert float(torch.linalg.matrix_norm(q.T.contiguous() @ q - eye)) <= 50 * n * u
    # Q block-triangularises A^T (the library reads the buffer column-major)
    t = q.T.contiguous() @ a.T.contiguous() @ q
    low = torch.linalg.matrix_norm(torch.tril(t, -2)) / torch.linalg.matrix_norm(a)
    assert float(low) <= 20 * n * u
