"""Work lists of short launches (host only): a list with fewer items than the
device has CUs is cut into shorter items, a long one is not, and every list
still covers its grids (the address walk checks each item's accesses, single
writers and that everything read is formed)."""

import pytest

from paper_1110_1616_amd import amr as A


def _single(n, dtype):
    p = A.make_params(len(n), n, 1, 2, 4, dtype)
    return p, A.make_grids([(0, (0,) * len(n), n)])


@pytest.mark.parametrize("n", [(2, 2, 2), (5, 9, 3), (14, 14, 1), (15, 14, 17), (37, 33, 35), (16, 16, 300)])
def test_short_lists_are_cut_and_cover_the_grid(n):
    p, g = _single(n, "f64")
    stats = A.amr_validate(p, g)
    # the lists of bands 2..4, once each for the batched, per-grid and explicit
    # band paths, and the adjoint's band-2 one: none longer than one item a CU
    # unless an item is a single plane already
    assert stats["flux_items"] <= 256 * 9
    for es in (4, 8, 16):
        loads, stores, reads = A.amr_selfcheck_addressing(p, g, es)
        assert loads > 0 and stores > 0 and reads > 0


def test_long_list_keeps_its_chunks():
    n = (160, 160, 160)
    p, g = _single(n, "f32")
    # band 2: 162 planes in chunks of at most 16 (11 of them), 11 x 11 tiles
    assert A.amr_validate(p, g)["flux_items"] >= 11 * 121
