"""The tridiagonal reduction's tagged exchange shares its memory with the plain
values that launches with larger tiles exchange, so no value may look like a
written word.  Kernel matrices have entries of every magnitude down to zero,
denormal floats among them, whose bit patterns are small integers."""

import numpy as np
import pytest

MAX_ORDER = 4225


def test_no_value_looks_like_a_written_word():
    from paper_2607_12430_amd import _lib
    tag = _lib.lib().msqrt_test_sytrd_tag
    tags = np.array([tag(j) for j in range(MAX_ORDER)], np.uint32)
    assert len(set(tags.tolist())) == MAX_ORDER
    # no finite float, alone in the upper half of a word ...
    assert np.isnan(tags.view(np.float32)).all()
    # ... and no finite double, whatever its lower half
    for low in (0, 1, 0x80000000, 0xFFFFFFFF):
        word = (tags.astype(np.uint64) << np.uint64(32)) | np.uint64(low)
        assert np.isnan(word.view(np.float64)).all()
    # nor a NaN that arithmetic makes (quiet, payload 0)
    assert not set(tags.tolist()) & {0x7FC00000, 0xFFC00000, 0x7FF80000, 0xFFF80000}


@pytest.mark.parametrize("prec,word", [("fp32", 1), ("fp64", 2)])
def test_exchange_memory_is_that_of_the_tiles_in_use(prec, word):
    """Two buffers of TR partial products, a column, a scalar and 64 bytes of sums
    per workgroup and diagonal workgroup; with at least 64 rows to a tile TR is
    at most n / 64 (not the 22 of the largest order), and at least one buffer of
    the largest tiles' layout has to be there."""
    from paper_2607_12430_amd import _lib
    size = _lib.lib().msqrt_test_sytrd_exchange

    def layout(n, tr):
        return 2 * 8 * (tr * n * word + n * word + word + 8 * tr * (tr + 1) // 2 + 8 * tr)

    for n in (193, 257, 300, 400, 512, 700, 1000, 1408, 1409, 2500, 4225):
        for batch in (1, 2, 64, 1000):
            got = size(_lib.PREC_NAMES[prec], n, batch, 256)
            if prec == "fp32" and n <= 256:
                assert got == 0  # the one-workgroup tail exchanges nothing
                continue
            assert layout(n, -(-n // 256)) <= got <= layout(n, min(22, -(-n // 64))), (n, batch)


def _kernel_matrix(n, length, nugget):
    x = np.arange(n)
    return np.exp(-((x[:, None] - x[None, :]) / length) ** 2 / 2) + nugget * np.eye(n)


# 64-row tiles follow larger ones where at most 22 of them cover the rest
# (1408 rows): right at the first column after, and far down.
@pytest.mark.gpu
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("n,length,nugget", [(1409, 3.0, 1e-2), (1472, 4.1, 1.0), (1536, 5.24, 1.0), (1536, 5.75, 0.1),
                                             (2049, 3.3, 1.0), (4096, 5.0, 0.1)])
def test_kernel_matrix(prec, n, length, nugget):
    import paper_2607_12430_amd as msq
    from scipy.linalg import eigvalsh_tridiagonal
    a = _kernel_matrix(n, length, nugget)
    if prec == "fp32":
        a = a.astype(np.float32).astype(np.float64)
    print(f"[tridiag exchange] {prec} n={n} length={length} nugget={nugget}", flush=True)
    d, e, _ = msq.test_sytrd(a, prec=prec)
    lam = np.linalg.eigvalsh(a)
    got = eigvalsh_tridiagonal(d.astype(np.float64), e.astype(np.float64))
    u = 2.0 ** -24 if prec == "fp32" else 2.0 ** -53
    # backward error of a Householder reduction: a modest multiple of n u
    assert np.max(np.abs(got - lam)) <= 2 * n * u * np.max(np.abs(lam))


# The same change of tiles for dense matrices, from 192- over 128- to 64-row tiles
# in one reduction, and the largest order (256-row tiles first).
@pytest.mark.gpu
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("n", [1409, 1500, 2900, 4225])
def test_dense(prec, n):
    import paper_2607_12430_amd as msq
    from scipy.linalg import eigvalsh_tridiagonal
    a = np.random.default_rng(n).standard_normal((n, n))
    a = a + a.T
    if prec == "fp32":
        a = a.astype(np.float32).astype(np.float64)
    print(f"[tridiag exchange] {prec} n={n} dense", flush=True)
    d, e, _ = msq.test_sytrd(a, prec=prec)
    lam = np.linalg.eigvalsh(a)
    got = eigvalsh_tridiagonal(d.astype(np.float64), e.astype(np.float64))
    u = 2.0 ** -24 if prec == "fp32" else 2.0 ** -53
    assert np.max(np.abs(got - lam)) <= 2 * n * u * np.max(np.abs(lam))
