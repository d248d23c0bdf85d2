"""Units of the Riemann solver (host only): its flux scales with the units of
density and velocity over the range that the wave speeds' squares leave.

Scaling rho by D, v by V, p by D V^2 and B by V sqrt(D) with powers of two (D
of four) scales every term of the solver exactly, so the fluxes of the scaled
states, scaled back, differ from the unscaled ones only where a value leaves
the normal range.  Small residuals do in FP32: each is below 2^-126 of its unit
and is summed with terms of order one unit, so 64 roundings are allowed."""

import ctypes as C

import numpy as np
import pytest

from paper_1110_1616_amd import amr as A

GAMMA = 5.0 / 3.0


def hlld(elem_bytes, states):
    s = np.ascontiguousarray(states, dtype=np.float64)
    f = np.empty((len(s), 7))
    fn = A.lib().amr_selfcheck_hlld
    fn.restype = C.c_int32
    fn.argtypes = [C.c_int32, C.c_int64, C.c_void_p, C.c_double, C.c_void_p]
    assert fn(elem_bytes, len(s), s.ctypes.data, GAMMA, f.ctypes.data) == A.AMR_OK
    return f


def states(n, seed, drift=1.0):
    r = np.random.default_rng(seed)
    s = np.zeros((n, 17))
    for o in (0, 8):
        s[:, o] = r.uniform(0.3, 3.0, n)
        s[:, o + 1:o + 4] = r.normal(0.0, drift, (n, 3))
        s[:, o + 4] = r.uniform(0.2, 2.0, n)
        s[:, o + 6:o + 8] = r.normal(0.0, 0.7, (n, 2))
    s[:, 16] = r.normal(0.0, 0.7, n)
    return s.astype(np.float32).astype(np.float64)


def scaled_error(elem_bytes, log4_rho, log2_v, s):
    D, V = 4.0 ** log4_rho, 2.0 ** log2_v
    B = V * 2.0 ** log4_rho
    u = np.array([D, V, V, V, D * V * V, B, B, B])
    t = s * np.concatenate([u, u, [B]])
    back = np.array([D * V, D * V * V, D * V * V, D * V * V, D * V ** 3, B * V, B * V])
    f, g = hlld(elem_bytes, s), hlld(elem_bytes, t) / back
    assert np.all(np.isfinite(g)), (log4_rho, log2_v)
    return np.max(np.abs(f - g) / (1.0 + np.abs(f)))


# (log4 of the density's unit, log2 of the velocity's): equal density and
# pressure from 1e-20 to 1e19 and 1e-30 at 1e6 in FP32, to 1e-240 and 1e240 in
# FP64, and velocities whose fourth power is still in range
@pytest.mark.parametrize("elem_bytes,units", [
    (4, [(-33, 0), (-31, 0), (-20, 0), (20, 0), (30, 0), (31, 0), (-50, 20), (-46, 20), (0, 14), (0, -14), (20, -14)]),
    (8, [(-400, 0), (-260, 0), (-240, 0), (240, 0), (256, 0), (400, 0), (-400, 120), (0, 120), (0, -120),
         (300, 120)]),
])
def test_flux_scales_with_the_units(elem_bytes, units):
    s = np.concatenate([states(1500, 3), states(500, 4, drift=0.1), states(500, 5, drift=4.0)])
    tol = 64 * (2.0 ** -24 if elem_bytes == 4 else 2.0 ** -53)
    for d, v in units:
        assert scaled_error(elem_bytes, d, v, s) <= tol, (d, v)
