"""The 64 x 64-tile GEMMs, which products with few 128-tiles take, at the edges
of their tiles (64 rows or columns), slabs (64 floats, 32 doubles of k) and
8-deep MFMA steps: |C - AB| <= 4 k u |A||B| element by element against a
float64 product in float, and a product of integer matrices in double, whose
sums are exact."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ta,tb", [(False, False), (True, False), (False, True), (True, True)])
@pytest.mark.parametrize("m,n,k", [(1, 1, 1), (63, 65, 7), (64, 64, 64), (65, 63, 65), (128, 1, 129),
                                   (200, 333, 8), (257, 190, 72), (1000, 501, 191)])
def test_float(ta, tb, m, n, k):
    import paper_2607_12430_amd as msq
    rng = np.random.default_rng(m + 3 * n + 7 * k + 11 * ta + 13 * tb)
    a = rng.standard_normal((k, m) if ta else (m, k)).astype(np.float32)
    b = rng.standard_normal((n, k) if tb else (k, n)).astype(np.float32)
    a64 = a.astype(np.float64).T if ta else a.astype(np.float64)
    b64 = b.astype(np.float64).T if tb else b.astype(np.float64)
    scale = np.abs(a64) @ np.abs(b64)
    print(f"[narrow gemm] float {m} {n} {k} {ta} {tb}", flush=True)
    c = msq.test_gemm_f32(a, b, split=False, ta=ta, tb=tb).astype(np.float64)
    assert np.all(np.abs(c - a64 @ b64) <= 4.0 * k * 2.0 ** -24 * scale)


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("n,k", [(1, 3), (63, 31), (64, 32), (65, 33), (130, 100), (1001, 40)])
def test_symmetric_output(prec, n, k):
    import paper_2607_12430_amd as msq
    rng = np.random.default_rng(n + 5 * k)
    # products of integers below 2^4 over fewer than 2^7 terms are exact in float too
    a = rng.integers(-15, 16, (n, k)).astype(np.float32 if prec == "fp32" else np.float64)
    print(f"[narrow gemm] symmetric {prec} {n} {k}", flush=True)
    c = msq.test_syrk(a, prec=prec).astype(np.float64)
    a64 = a.astype(np.float64)
    assert np.array_equal(c, a64 @ a64.T)


@pytest.mark.parametrize("ta,tb", [(False, False), (True, False), (False, True), (True, True)])
@pytest.mark.parametrize("m,n,k", [(1, 1, 1), (63, 65, 7), (64, 64, 64), (65, 63, 65), (200, 333, 17),
                                   (257, 190, 72), (1000, 501, 191)])
def test_bf16_split(ta, tb, m, n, k):
    import torch
    import paper_2607_12430_amd as msq
    rng = np.random.default_rng(m + 3 * n + 7 * k + 11 * ta + 13 * tb)
    a = rng.standard_normal((k, m) if ta else (m, k)).astype(np.float32)
    b = rng.standard_normal((n, k) if tb else (k, n)).astype(np.float32)
    a64 = a.astype(np.float64).T if ta else a.astype(np.float64)
    b64 = b.astype(np.float64).T if tb else b.astype(np.float64)
    def parts(x):
        t = torch.from_numpy(np.ascontiguousarray(x.astype(np.float32)))
        hi = t.to(torch.bfloat16).float()
        return hi.double().numpy(), (t - hi).to(torch.bfloat16).double().numpy()

    ah, al = parts(a64)
    bh, bl = parts(b64)
    ref = ah @ bh + ah @ bl + al @ bh
    scale = np.abs(a64) @ np.abs(b64)
    print(f"[narrow gemm] split {m} {n} {k} {ta} {tb}", flush=True)
    c = msq.test_gemm_f32(a, b, split=True, ta=ta, tb=tb).astype(np.float64)
    # what the split product is in exact arithmetic, summed in float
    assert np.all(np.abs(c - ref) <= 4.0 * 3 * k * 2.0 ** -24 * scale)
