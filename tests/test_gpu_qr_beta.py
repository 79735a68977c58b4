"""The entry that a reflector of the real QR writes in place of a column, beta =
-sign(x_0) ||x||.  Every bulge replaces the subdiagonal entry that it passes by
such a norm, so a mean error of the norms is a drift of the subdiagonal: n
bulges add it up n times, where errors of mean zero add up to sqrt(n) of one."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,bits", [("fp32", 24), ("fp64", 53)])
def test_beta_has_no_drift(prec, bits):
    """Rounding to nearest leaves errors of at most one unit roundoff or two with
    mean zero: over 2^20 vectors their mean is within 2 / 2^10 of one, at five
    standard deviations within 0.01."""
    import paper_2607_12430_amd as msq
    r = np.random.default_rng(3)
    x = r.standard_normal((1 << 20, 4))
    x[:, 1:] *= 10.0 ** r.uniform(-2, 2, (len(x), 1))  # either entry may dominate
    x[::3, 2] = 0.0
    x *= 10.0 ** r.uniform(-3, 3, (len(x), 1))
    if prec == "fp32":
        x = x.astype(np.float32).astype(np.float64)
    print(f"[qr beta] {prec}", flush=True)
    beta = msq.test_qr_beta(x, prec)
    e = x[:, :3].astype(np.longdouble)
    ref = -np.copysign(np.sqrt((e * e).sum(1)), e[:, 0])
    err = (((beta - ref) / ref) * np.longdouble(2.0) ** bits).astype(float)
    print(f"[qr beta] {prec}: mean {err.mean():.4f}, rms {np.sqrt((err ** 2).mean()):.3f}, "
          f"largest {np.abs(err).max():.2f} units", flush=True)
    assert np.abs(err).max() <= 4.0
    assert abs(err.mean()) <= 0.01
