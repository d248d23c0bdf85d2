"""The address walk of the fused kernel covers what the kernel loads: every lane
of every item loads a (clamped) cell of each plane, also lanes outside the grid
(host only)."""

import pytest

from paper_1110_1616_amd import amr as A


@pytest.mark.parametrize("n", [(6, 5, 4), (20, 18, 16), (64, 48)])
def test_every_lane_of_a_fused_item_is_walked(n):
    nd = len(n)
    p = A.make_params(nd, n, 1, 2, 4)
    grids = A.make_grids([(0, (0,) * nd, n)])
    loads, stores, reads = A.amr_selfcheck_addressing(p, grids, 8)
    # a fused item is a column of at least one updated plane; with the planes
    # below and above it a lane loads four of them, each with its high faces
    items = A.amr_validate(p, grids)["flux_items"]  # the flux lists' tiles overlap less: no more than the fused ones
    assert loads >= items * 256 * (4 * 4 if nd == 3 else 3), (loads, items)
