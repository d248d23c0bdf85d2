"""The configuration a new hierarchy reports is the one it runs, so setting back
what was read changes neither."""

import pytest
import torch

from paper_1110_1616_amd import amr as A
from paper_1110_1616_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("emf,mode", [(A.AMR_EMF_MEAN, 8), (A.AMR_EMF_UPWIND, 0)])
@pytest.mark.parametrize("n", [(48, 40), (20, 18, 16)])
def test_setting_back_the_reported_configuration_changes_nothing(n, emf, mode):
    nd = len(n)
    ic = I.smooth_mhd(nd, n, seed=3)
    H = A.Hierarchy(nd, n, [(0, (0,) * nd, n)], ghost=4, dx0=ic["dx"], emf=emf)
    U, V = H.new_state(), H.new_state()
    H.load_primitive(U, 0, ic["prim"], ic["b"])
    H.fill(0, A.AMR_FILL_SAME_LEVEL, U)
    H.compute_dt(U)

    def step():
        """Results, and whether the two kernels ran: they pass every face flux
        through the workspace, where the fused one leaves nothing on one grid."""
        H.ws.zero_()
        H.advance(U, V, cycle=0, band=4)
        assert H.error_flags()[0] == 0
        return [f.clone() for f in V.fields], bool(H.ws.any())

    assert A.amr_get_launch_config(H.h) == (1, 16, mode)
    want, two = step()
    assert two == (mode == 0)
    H.set_launch_config(*A.amr_get_launch_config(H.h))
    got, again = step()
    assert again == two
    assert A.amr_get_launch_config(H.h) == (1, 16, mode)
    for a, b in zip(got, want):
        assert torch.equal(a, b)
