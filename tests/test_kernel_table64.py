"""The FP64 kernel tables (swim_kernel_eval_host in FP64: the tables' own code on
the host) against the closed forms in 60 digits, relative to each function
itself from near contact on: Ht = H1 - H1(0) vanishes like r^2 there, so a
coordinate that has lost the low bits of r^2 shows (5e-13 at 0.01 eps).

Bars: the direct evaluation of the closed forms is within 7e-16 (Ht) below
0.3 eps; the table adds the quotient by its coordinate, the transform to
coefficients and a Horner step, each about one rounding (1.1e-16): 1.5e-15."""
import mpmath as mp
import numpy as np
import pytest

from paper_1910_12007_amd import swim


def _reading(alpha, eps, t):
    """Ht, H2 of the reading's blob (alpha = 0: the Stokes closed form)."""
    alpha, eps, t = mp.mpf(alpha), mp.mpf(eps), mp.mpf(t)
    d = t / eps ** 2
    if alpha == 0:
        L = mp.log1p(d)
        return (L / d - 1 - L) / (8 * mp.pi), (1 - L / d) / (4 * mp.pi * t)
    z0, z = alpha * eps, alpha * mp.sqrt(t + eps ** 2)
    c = 1 / (z0 * mp.besselk(1, z0))
    g, g0 = (-c * mp.besselk(0, q) / (2 * mp.pi) for q in (z, z0))
    M = c * (z * mp.besselk(1, z) - z0 * mp.besselk(1, z0)) / (2 * mp.pi * alpha ** 2)
    return M / t - g + g0 / 2, (g - 2 * M / t) / t


@pytest.mark.parametrize("alpha", [0.0, 0.5, 10.0])
@pytest.mark.parametrize("N", [64, 512])
def test_relative_accuracy_to_contact(alpha, N):
    mp.mp.dps = 60
    eps = 1.5 / (N - 1)
    # both sides of the first interval's end (v = 17/16) and of v = 2 among them
    s = 4.0 ** np.ceil(-np.log2(eps) - 1e-12)
    edges = np.sqrt(np.array([1.0 / 16, 1.0]) / s)
    r = np.concatenate([eps * np.geomspace(1e-6, 0.3, 60), edges * (1 - 1e-9), edges * (1 + 1e-9)])
    r = r[r <= 0.3 * eps]
    h, g, _ = swim.swim_kernel_eval_host(swim.SWIM_F64, alpha, eps, r * r, blob=swim.SWIM_BLOB_READING)
    for i in range(len(r)):
        a, b = _reading(alpha, eps, (r * r)[i])
        assert abs(float((mp.mpf(h[i]) - a) / a)) < 1.5e-15, (r[i] / eps, h[i], float(a))
        assert abs(float((mp.mpf(g[i]) - b) / b)) < 1.5e-15, (r[i] / eps, g[i], float(b))


@pytest.mark.parametrize("blob", [swim.SWIM_BLOB_READING, swim.SWIM_BLOB_PAPER])
@pytest.mark.parametrize("alpha", [0.0, 1.3])
def test_continuous_over_interval_edges(blob, alpha):
    """Values on either side of every interval's end, one FP64 step apart, agree
    to the same bar on the function's scale (|Ht|, and H2 by its value)."""
    eps = 1.5 / 63
    s = 4.0 ** np.ceil(-np.log2(eps) - 1e-12)
    v = np.array([2.0 ** e * (1 + (j + 1) / 16) for e in range(30) for j in range(16)])
    t = (v - 1) / s
    lo, hi = (swim.swim_kernel_eval_host(swim.SWIM_F64, alpha, eps, q, blob=blob) for q in (np.nextafter(t, 0), t))
    scale = np.maximum(np.abs(hi[0]) + t * np.abs(hi[1]), 1e-300)
    # the step itself moves t by 2^-52 of its value at most, and both functions
    # change by less than their scale per unit of ln t
    bar = 2 * 1.5e-15 + 2.0 ** -51
    assert np.max(np.abs(hi[0] - lo[0]) / scale) < bar
    assert np.max(t * np.abs(hi[1] - lo[1]) / scale) < bar


def test_zero_distance():
    for blob in (swim.SWIM_BLOB_READING, swim.SWIM_BLOB_PAPER):
        for alpha in (0.0, 2.0):
            h, g, _ = swim.swim_kernel_eval_host(swim.SWIM_F64, alpha, 0.02, np.array([0.0, 1e-300, 1e-30]), blob=blob)
            assert h[0] == 0.0 and np.all(np.isfinite(h)) and np.all(np.isfinite(g))
            # Ht is proportional to t, H2 constant
            assert abs(h[2] / h[1] / 1e270 - 1) < 1e-12 and g[0] == g[1] and abs(g[2] / g[0] - 1) < 1e-12


@pytest.mark.parametrize("alpha", [2.0, 80.0])
@pytest.mark.parametrize("e", [-250, -200, 200, 250])
def test_scale_invariance(alpha, e):
    """The paper blob's values depend on alpha eps and r / eps alone (H2 times a
    length squared): in units 2^e times as long, every operation scales exactly."""
    eps, s = 0.0125, 2.0 ** e
    t = (np.geomspace(1e-3, 1e9, 60) * eps) ** 2
    h0, g0, _ = swim.swim_kernel_eval_host(swim.SWIM_F64, alpha, eps, t, blob=swim.SWIM_BLOB_PAPER)
    h, g, _ = swim.swim_kernel_eval_host(swim.SWIM_F64, alpha / s, eps * s, t * s * s, blob=swim.SWIM_BLOB_PAPER)
    assert np.array_equal(h, h0) and np.array_equal(g * s * s, g0)
