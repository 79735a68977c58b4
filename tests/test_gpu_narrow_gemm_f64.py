"""The double GEMM with 64 x 64 tiles, every operand order, as a batch, with a C
that is added to (the last tile of a row or column overlaps the one before: no
element may be counted twice) and with a shorter last entry.  Integer matrices,
whose sums are exact."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

ORDERS = [(False, False), (True, False), (False, True), (True, True)]


def _ints(shape, rng):
    return rng.integers(-9, 10, shape).astype(np.float64)


def _op(x, t):
    return np.swapaxes(x, 1, 2) if t else x


@pytest.mark.parametrize("ta,tb", ORDERS)
@pytest.mark.parametrize("k", [1, 31, 32, 33, 100])
@pytest.mark.parametrize("m,n", [(1, 1), (63, 64), (64, 65), (65, 63), (130, 200), (257, 70)])
def test_batch_added(ta, tb, m, n, k):
    import paper_2607_12430_amd as msq
    rng = np.random.default_rng(m + 7 * n + 31 * k)
    a = _ints((3, k, m) if ta else (3, m, k), rng)
    b = _ints((3, n, k) if tb else (3, k, n), rng)
    c = _ints((3, m, n), rng)
    print(f"[narrow gemm f64] {m} {n} {k} {ta} {tb}", flush=True)
    ref = _op(a, ta) @ _op(b, tb)
    assert np.array_equal(msq.test_gemm_f64(a, b, ta=ta, tb=tb), ref)
    assert np.array_equal(msq.test_gemm_f64(a, b, c, ta=ta, tb=tb), ref + c)


@pytest.mark.parametrize("ta,tb", ORDERS)
@pytest.mark.parametrize("k,k_last", [(64, 1), (64, 33), (100, 99), (33, 32)])
def test_shorter_last_entry(ta, tb, k, k_last):
    import paper_2607_12430_amd as msq
    rng = np.random.default_rng(k + 7 * k_last)
    m, n = 65, 130
    a = _ints((4, k, m) if ta else (4, m, k), rng)
    b = _ints((4, n, k) if tb else (4, k, n), rng)
    print(f"[narrow gemm f64] split {k} {k_last} {ta} {tb}", flush=True)
    got = msq.test_gemm_f64(a, b, ta=ta, tb=tb, k_last=k_last)
    ref = _op(a, ta) @ _op(b, tb)
    ref[-1] = _op(a, ta)[-1][:, :k_last] @ _op(b, tb)[-1][:k_last]
    assert np.array_equal(got, ref)
