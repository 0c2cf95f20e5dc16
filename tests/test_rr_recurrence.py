"""r.r of the updated residual from the sums of one meeting,

    |r - a q|^2 = r.r - 2 a (r.q) + a^2 (q.q),

(the device's next_rr) against the sum over the residual as it is stored, on
CG iterations replayed on the CPU with the device's roundings: vectors in the
working precision, one rounding per update, sums in FP64.

The bounds are derived, not measured.  The formula is used where the result
exceeds a hundredth of a^2 q.q; then a^2 q.q < 100, r.r < 121 and 2 a r.q < 220
times the result, and with sums that are right to 18 rounding errors of 2^-53
the result is right to 441 * 18 * 2^-53 < 1e-12.  An FP32 residual is rounded
after the update, each entry by at most 2^-24 of itself, so r.r changes by at
most 2^-23 of itself; for roundings that are independent and entries of one
size the change has a standard deviation below 2^-23 / L, five of which are
allowed here."""

import numpy as np
import pytest
import scipy.fft as sf

from workloads import spectrum, padded_instance, periodic_instance


def _next_rr(t, a):
    """(result, whether the device uses it) from t = p.q, r.r, r.q, q.q."""
    rr = a * (a * t[3] - 2.0 * t[2]) + t[1]
    return rr, rr > 0.01 * (a * a * t[3])


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("L,padded,eps", [(16, 1, 1e-3), (32, 0, 1e-2), (32, 1, 1e-4), (64, 1, 1e-3), (128, 1, 1e-4)])
def test_error_of_the_formula(L, padded, eps, dtype):
    inst = (padded_instance if padded else periodic_instance)(L, [41, L, padded], eps=eps)
    g = inst["ghat"].astype(dtype)
    d = inst["d"].astype(dtype)
    M = g.shape[0]

    def apply(p):
        z = np.zeros((M, M), dtype)
        z[:L, :L] = p
        return (d * p + np.real(sf.ifft2(sf.fft2(z) * g))[:L, :L].astype(dtype)).astype(dtype)

    def dot(u, v):
        return float(np.sum(u.astype(np.float64) * v.astype(np.float64)))

    r = inst["b"].astype(dtype)
    p = r.copy()
    worst, used = 0.0, 0
    for _ in range(60):
        q = apply(p)
        t = [dot(p, q), dot(r, r), dot(r, q), dot(q, q)]
        a = dtype(t[1] / t[0])
        # (a multiply-add in the working precision rounds once)
        r = (r.astype(np.longdouble) - np.longdouble(a) * q.astype(np.longdouble)).astype(dtype)
        rr, sure = _next_rr(t, float(a))
        direct = dot(r, r)
        if sure:
            used += 1
            worst = max(worst, abs(rr - direct) / direct)
        p = (r.astype(np.longdouble) + np.longdouble(dtype(direct / t[1])) * p.astype(np.longdouble)).astype(dtype)
    print(L, padded, dtype.__name__, used, worst)
    assert used >= 50
    assert worst <= (1e-12 if dtype is np.float64 else 1e-12 + 5 * 2.0 ** -23 / L)
