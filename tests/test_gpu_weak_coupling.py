"""Blocks coupled by entries whose squares underflow: the reflector of a column
that holds nothing else must neither over- nor underflow.  Against the root of
the uncoupled blocks, from which the root differs by about the coupling."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _blocks(n, coupling, seed):
    r = np.random.default_rng(seed)
    h = n // 2
    a = np.zeros((n, n))
    x = r.standard_normal((h, h))
    y = r.standard_normal((n - h, n - h))
    a[:h, :h] = x @ x.T / h + np.eye(h)
    a[h:, h:] = y @ y.T / (n - h) + np.eye(n - h)
    a = 0.5 * (a + a.T)
    a[:h, h:] = coupling * r.uniform(0.5, 1.0, (h, n - h))
    a[h:, :h] = a[:h, h:].T
    return a


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("n", [20, 90, 300, 600])
@pytest.mark.parametrize("coupling", [1e-20, 1e-40, 1e-44, 1e-100, 1e-139, 1e-150, 1e-155, 1e-158, 1e-161, 1e-170, 1e-300])
def test_spd(prec, n, coupling):
    import torch
    import paper_2607_12430_amd as msq
    a = _blocks(n, coupling, n)
    print(f"[weak coupling] spd {prec} n={n} {coupling}", flush=True)
    d, e, _ = msq.test_sytrd(a, prec=prec)
    assert np.isfinite(d).all() and np.isfinite(e).all()
    x, info = msq.sqrtm(torch.from_numpy(a).cuda(), prec=prec, structure="hpd", fallback=False)
    assert info["status"] == "ok" and info["relres"] <= 1e-13
    lam, q = np.linalg.eigh(_blocks(n, 0.0, n))
    root = (q * np.sqrt(lam)) @ q.T
    assert np.linalg.norm(x.cpu().numpy() - root) <= 1e-12 * np.linalg.norm(root)


def _general(n, coupling, seed, cplx):
    r = np.random.default_rng(seed)
    h = n // 2
    a = r.standard_normal((n, n)) / np.sqrt(n)
    if cplx:
        a = a + 1j * r.standard_normal((n, n)) / np.sqrt(n)
    a = a + 3.0 * np.eye(n)
    a[h:, :h] *= coupling
    return a


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("n", [20, 90, 300])
@pytest.mark.parametrize("coupling", [1e-10, 1e-17, 1e-19, 1e-21, 1e-22, 1e-30, 1e-44, 1e-100, 1e-150, 1e-160, 1e-162, 1e-300])
def test_complex_hessenberg(prec, n, coupling):
    import paper_2607_12430_amd as msq
    a = _general(n, coupling, n, True)
    print(f"[weak coupling] hessenberg {prec} n={n} {coupling}", flush=True)
    h, q = msq.test_gehrd(a, prec)
    u = 2.0 ** -24 if prec == "fp32" else 2.0 ** -53
    # n reflections, each with an error of a few u in Frobenius norm
    assert np.linalg.norm(q.conj().T @ q - np.eye(n)) <= 10 * n * u
    assert np.linalg.norm(q @ h @ q.conj().T - a) <= 10 * n * u * np.linalg.norm(a)


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("n", [20, 90, 300])
@pytest.mark.parametrize("coupling", [1e-10, 1e-17, 1e-19, 1e-21, 1e-22, 1e-30, 1e-44, 1e-100, 1e-150, 1e-160, 1e-162, 1e-300])
@pytest.mark.parametrize("cplx", [False, True])
def test_general_root(prec, n, coupling, cplx):
    import torch
    import paper_2607_12430_amd as msq
    a = _general(n, coupling, n, cplx)
    print(f"[weak coupling] root {prec} n={n} {coupling} {cplx}", flush=True)
    f = msq.factor(torch.from_numpy(a).cuda(), prec=prec, structure="general")
    if not cplx:
        q = f.export(prec == "fp32", "general")[0][0].astype(np.float64)
        u = 2.0 ** -24 if prec == "fp32" else 2.0 ** -53
        # the Hessenberg reduction's and that of about 2 n QR sweeps of n rows
        assert np.linalg.norm(q.T @ q - np.eye(n)) <= 30 * n * u
    f.close()
    x, info = msq.sqrtm(torch.from_numpy(a).cuda(), prec=prec, structure="general", fallback=False)
    assert info["status"] == "ok" and info["relres"] <= 1e-13
    assert info["steps"] <= (3 if prec == "fp32" else 1)
