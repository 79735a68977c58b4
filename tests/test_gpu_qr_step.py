"""The elementary transformations of the shifted QR: a sweep applies each of
them to every row of Z and to most of H, so an error in their normalisation is
the same everywhere and adds up over the sweeps, unlike the rounding of the
single entries.  They are orthogonal (unitary) far beyond the working
precision, checked here in exact rational arithmetic."""

from fractions import Fraction as F

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _vectors(m, seed):
    r = np.random.default_rng(seed)
    x = r.standard_normal((m, 4))
    # graded entries, zeros, ties, large and small scales
    x[::5] *= 10.0 ** r.uniform(-12, 0, (len(x[::5]), 4))
    x[::7] *= 10.0 ** r.uniform(-20, 15, (len(x[::7]), 1))
    x[1::11, 2] = 0.0
    x[2::13, 1:] = x[2::13, :1]
    return x


@pytest.mark.parametrize("prec,digits", [("fp32", 42), ("fp64", 98)])
def test_reflector_is_orthogonal(prec, digits):
    """(tau + tl) v^T v = 2: tau's relative error is at most 2^-22 (an estimate
    of one unit in the last place and its rounding) in float and 2^-52 in
    double; tl removes it to first order and is itself rounded, so what is left
    is below 2^-43 and 2^-99."""
    import paper_2607_12430_amd as msq
    x = _vectors(3000, 1)
    print(f"[qr step] reflectors {prec}", flush=True)
    for tau, tl, w1, w2 in msq.test_qr_step(x, False, prec):
        assert tau != 0.0 and max(abs(w1), abs(w2)) <= 1.0 + 2.0 ** -20
        n2 = 1 + F(w1) ** 2 + F(w2) ** 2
        assert abs((F(tau) + F(tl)) * n2 - 2) <= F(1, 2 ** digits), (tau, tl, w1, w2)


def test_rotation_is_unitary():
    """(1 + h)^2 (c^2 + |s|^2) = 1 in double: the sum is off by at most 2^-50 (a
    handful of roundings), h removes that to first order and is rounded: 2^-99.
    In float h is zero and the sum is within 2^-20."""
    import paper_2607_12430_amd as msq
    x = _vectors(3000, 2)
    print("[qr step] rotations", flush=True)
    for c, sr, si, h in msq.test_qr_step(x, True, "fp64"):
        n2 = F(c) ** 2 + F(sr) ** 2 + F(si) ** 2
        assert abs((1 + F(h)) ** 2 * n2 - 1) <= F(1, 2 ** 97), (c, sr, si, h)
    for c, sr, si, h in msq.test_qr_step(x, True, "fp32"):
        n2 = F(c) ** 2 + F(sr) ** 2 + F(si) ** 2
        assert h == 0.0 and abs(n2 - 1) <= F(1, 2 ** 20)
