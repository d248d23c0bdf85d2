"""What cancels between the z-faces of a cell cancels in the update.

A state that does not depend on z has the same fluxes through both z-faces of a
cell, among them a pressure (m_z) and an E_x, E_y of a strong B_z carried along
(B_x, B_y) far larger than the fields they act on.  The differences are exactly
zero, so in FP32 those fields keep the rounding of their own size: four steps of
some tens of roundings each, 256 x 2^-24 of the largest value.  (A pressure term
rounded on its own is 2^-24 x dt/dz x p here, 1e4 roundings of m_z.)"""

import numpy as np
import pytest

import oracle as O
from gpu_util import log
from paper_1110_1616_amd import amr as A

pytestmark = pytest.mark.gpu

GAMMA = 5.0 / 3.0
EPS = 1e-5


@pytest.mark.parametrize("launch", [(1, 16, 0), (1, 16, 8), (1, 4, 12)])
def test_small_fields_keep_their_digits_next_to_uniform_z_fluxes(launch):
    n = (20, 18, 12)
    x, y, z = [(np.arange(m) + 0.5) / m for m in n]
    X, Y, Z = x[None, None, :], y[None, :, None], z[:, None, None]
    one = np.ones((n[2], n[1], n[0]))
    prim = [one, 0.05 * one, 0.04 * one, EPS * np.sin(2 * np.pi * (X + Y)) + 0.0 * Z, one]
    b = [np.broadcast_to(EPS * np.cos(2 * np.pi * Y), (n[2], n[1], n[0] + 1)),
         np.broadcast_to(EPS * np.sin(2 * np.pi * X), (n[2], n[1] + 1, n[0])), np.ones((n[2] + 1, n[1], n[0]))]
    f32 = [np.ascontiguousarray(np.float32(a), dtype=np.float64) for a in prim + b]
    ic = {"ndim": 3, "n": n, "dx": [1.0 / m for m in n], "prim": f32[:5], "b": f32[5:]}
    dts = [0.005] * 4
    want, _ = O.uniform_run(ic, GAMMA, 0.4, 4, g=4, fill_every=2, dts=dts)
    H = A.Hierarchy(3, n, [(0, (0, 0, 0), n)], ghost=4, dtype="f32", dx0=ic["dx"], gamma=GAMMA)
    H.set_launch_config(*launch)
    U, V = H.new_state(), H.new_state()
    H.load_primitive(U, 0, ic["prim"], ic["b"])
    for s, dt in enumerate(dts):
        if s % 2 == 0:
            H.fill(0, A.AMR_FILL_SAME_LEVEL, U)
        H.dt0.fill_(dt)
        H.advance(U, V, cycle=0, band=4 - 2 * (s % 2))
        U, V = V, U
    assert H.error_flags()[0] == 0
    got = dict(zip(A.FIELDS, zip(H.store_interior(U, 0), want)))
    for f in ("mz", "bx", "by"):
        a, w = got[f]
        err = np.max(np.abs(a - w)) / np.max(np.abs(w))
        log(f"launch {launch} {f}: {err:.1e}")
        assert err <= 256 * 2.0 ** -24, (f, err)
