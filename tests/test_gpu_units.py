"""The advance in other units of density and velocity: a state scaled by powers
of two (density by D, velocity by V, pressure by D V^2, field by V sqrt(D), the
step by 1 / V) evolves into the scaled state.

Every term of the scheme scales exactly, so the results differ at most where a
residual leaves the normal range: it is then below the smallest normal number
times a few, next to fields of one unit, and in FP32 units down to 4^-50 that is
2^-126 / 2^-100 = 2^-26 of the unit, half a rounding; four steps of a few dozen
such terms stay below 1e3 roundings of the largest value."""

import numpy as np
import pytest

from gpu_util import log
from paper_1110_1616_amd import amr as A
from paper_1110_1616_amd import inputs as I

pytestmark = pytest.mark.gpu

GAMMA = 5.0 / 3.0


def run(ic, n, dtype, launch, dts, log4_rho=0, log2_v=0):
    D, V = 4.0 ** log4_rho, 2.0 ** log2_v
    B = V * 2.0 ** log4_rho
    prim = [a * u for a, u in zip(ic["prim"], (D, V, V, V, D * V * V))]
    nd = len(n)
    H = A.Hierarchy(nd, n, [(0, (0,) * nd, n)], ghost=4, dtype=dtype, dx0=ic["dx"], gamma=GAMMA)
    H.set_launch_config(*launch)
    U, W = H.new_state(), H.new_state()
    H.load_primitive(U, 0, prim, [b * B for b in ic["b"]])
    for s, dt in enumerate(dts):
        if s % 2 == 0:
            H.fill(0, A.AMR_FILL_SAME_LEVEL, U)
        H.dt0.fill_(dt / V)
        H.advance(U, W, cycle=0, band=4 - 2 * (s % 2))
        U, W = W, U
    assert H.error_flags()[0] == 0
    units = (D, D * V, D * V, D * V, D * V * V, B, B, B)
    return [np.asarray(f) / u for f, u in zip(H.store_interior(U, 0), units)]


@pytest.mark.parametrize("launch", [(1, 16, 0), (1, 16, 8)])
@pytest.mark.parametrize("n", [(22, 17), (18, 13, 11)])
@pytest.mark.parametrize("dtype,units", [
    ("f32", [(-33, 0), (30, 0), (-50, 20), (0, 14)]),
    ("f64", [(-300, 0), (-240, 0), (300, 0), (0, 100)]),
])
def test_steps_scale_with_the_units(dtype, units, n, launch):
    ic = I.smooth_mhd(len(n), n, seed=21, v_rms=0.3, b_rms=0.4, jump=True)
    # FP32 inputs, so that both runs start from the same digits
    ic["prim"] = [np.float32(a).astype(np.float64) for a in ic["prim"]]
    ic["b"] = [np.float32(a).astype(np.float64) for a in ic["b"]]
    dts = [0.2 * min(ic["dx"][:len(n)]) / 4.0] * 4
    want = run(ic, n, dtype, launch, dts)
    tol = 1e3 * (2.0 ** -24 if dtype == "f32" else 2.0 ** -53)
    for d, v in units:
        log(f"case: {dtype} {n} launch {launch} log4 rho {d} log2 v {v}")
        got = run(ic, n, dtype, launch, dts, d, v)
        for f, a, b in zip(A.FIELDS, got, want):
            err = np.max(np.abs(a - b)) / max(np.max(np.abs(b)), 1e-3)
            assert err <= tol, (f, d, v, err)
