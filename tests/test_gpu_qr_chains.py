"""The chain QR of the general path at the orders where its windows, chains
and final blocks begin and end (windows of 128 / 96 / 96 / 64 rows for real
float, real double, complex float and complex double), and on inputs whose
shifts make no progress without exceptional sweeps."""

import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu

U_ROUND = {"fp32": 2.0 ** -24, "fp64": 2.0 ** -53}


def _matrix(kind, n, seed):
    rng = np.random.default_rng(seed)
    if kind == "random":
        return 2.0 * np.eye(n) + rng.standard_normal((n, n)) / np.sqrt(n)
    if kind == "cyclic":  # spectrum on a circle: every plain shift is symmetric to it
        return 3.0 * np.eye(n) + np.roll(np.eye(n), 1, axis=0)
    # real, clustered eigenvalues under a strictly upper part
    q = np.linalg.qr(rng.standard_normal((n, n)))[0]
    t = np.triu(rng.standard_normal((n, n)), 1) / n + np.diag(np.repeat([1.0, 2.0, 3.0, 4.0], (n + 3) // 4)[:n])
    return q @ t @ q.T


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("kind,n", [("random", 3), ("random", 96), ("random", 97), ("random", 128),
                                    ("random", 129), ("random", 193), ("random", 460),
                                    ("cluster", 230), ("cyclic", 150)])
def test_real_schur_form(prec, kind, n):
    import torch
    import paper_2607_12430_amd as msq
    a = _matrix(kind, n, n)
    print(f"[chains] real {prec} {kind} n={n}", flush=True)
    f = msq.factor(torch.from_numpy(a).cuda(), prec=prec, structure="general")
    q, s, k = f.export(single=prec == "fp32", structure="general")
    q, s = q[0].astype(np.float64), s[0].reshape(n, n).T.astype(np.float64)
    u = U_ROUND[prec]
    assert np.linalg.norm(q.T @ q - np.eye(n)) <= 50 * n * u
    assert np.all(np.tril(s, -2) == 0)
    assert np.all(np.diff(np.nonzero(np.diag(s, -1))[0]) >= 2)
    # the library factors A^T; the root adds n u |S| |S| to the Schur form's error
    at = a.T / 4.0 ** k
    tol = 20 * n * u * max(1.0, np.linalg.norm(s) ** 2 / np.linalg.norm(at))
    assert np.linalg.norm(q @ s @ s @ q.T - at) <= tol * np.linalg.norm(at)


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("kind,n", [("random", 2), ("random", 64), ("random", 65), ("random", 97),
                                    ("random", 161), ("random", 300), ("cluster", 130), ("cyclic", 110)])
def test_complex_schur_form(prec, kind, n):
    import paper_2607_12430_amd as msq
    rng = np.random.default_rng(n + 1)
    a = _matrix(kind, n, n).astype(np.complex128)
    if kind == "random":
        a = a + 1j * rng.standard_normal((n, n)) / np.sqrt(n)
    print(f"[chains] complex {prec} {kind} n={n}", flush=True)
    t, q = msq.test_schur(a, prec=prec)
    u = U_ROUND[prec]
    assert np.all(np.tril(t, -1) == 0)
    assert np.linalg.norm(q.conj().T @ q - np.eye(n)) <= 50 * n * u
    assert np.linalg.norm(q @ t @ q.conj().T - a) <= 20 * n * u * np.linalg.norm(a)


def test_real_root_with_exceptional_sweeps():
    import torch
    import paper_2607_12430_amd as msq
    a = _matrix("cyclic", 333, 0)
    x, info = msq.sqrtm(torch.from_numpy(a).cuda(), structure="general")
    assert info["status"] == "ok", info
    xh = x.cpu().numpy()
    assert O.relres(xh, a) <= 1e-13
    assert O.relerr(xh, O.sqrtm_real(a)) <= 1e-11
