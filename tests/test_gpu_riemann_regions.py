"""Every region of the Riemann solver's fan on the GPU, against the oracle.

A smooth 3-D state carried along the axes: at rest the inner (double-star)
states hold x/t = 0, at a drift between the Alfven and the fast speed the star
states do (either side, by its sign), and beyond the fast speed the outer
states.  Both kernels of the advance run (fused and flux + update).  Bounds:
the package's parity bars, 1e-10 in FP64; in FP32 the pressure is the
difference of E and a kinetic energy of up to 8 p, so 10 times the rounding of
a few steps, 10 x 4 x 6e-8 < 1e-5.
"""

import numpy as np
import pytest

import oracle as O
from gpu_util import log, normwise_errors
from paper_1110_1616_amd import amr as A
from paper_1110_1616_amd import inputs as I

pytestmark = pytest.mark.gpu

GAMMA = 5.0 / 3.0


@pytest.mark.parametrize("dtype,tol", [("f64", 1e-10), ("f32", 1e-5)])
@pytest.mark.parametrize("drift", [(0.0, 0.0, 0.0), (0.8, -0.8, 0.8), (-4.0, 4.0, 0.8), (4.0, -0.8, -4.0)])
def test_riemann_regions_match_oracle(drift, dtype, tol):
    n = (22, 17, 19)
    ic = I.smooth_mhd(3, n, seed=15, v_rms=0.1, b_rms=0.3)
    for a in range(3):
        ic["prim"][1 + a] = ic["prim"][1 + a] + drift[a]
    want, dts = O.uniform_run(ic, GAMMA, 0.4, 4, g=4, fill_every=2)
    for launch in ((1, 16, 0), (1, 16, 8)):
        log(f"case: drift {drift} {dtype} launch {launch}")
        H = A.Hierarchy(3, n, [(0, (0, 0, 0), n)], ghost=4, dtype=dtype, dx0=ic["dx"], gamma=GAMMA)
        H.set_launch_config(*launch)
        U, V = H.new_state(), H.new_state()
        H.load_primitive(U, 0, ic["prim"], ic["b"])
        for s, dt in enumerate(dts):
            if s % 2 == 0:
                H.fill(0, A.AMR_FILL_SAME_LEVEL, U)
            H.dt0.fill_(float(dt))
            H.advance(U, V, cycle=0, band=4 - 2 * (s % 2))
            U, V = V, U
        assert H.error_flags()[0] == 0
        err = normwise_errors(H.store_interior(U, 0), want)
        log(f"  errors per field: {err}")
        assert np.all(err <= tol), err
