"""How the batched launches are cut along z (host only): a list of fewer items
than the device has CUs into the shortest items that still have one each, a
longer one not at all, for the flux and the fused kernel's lists."""

import ctypes as C

import pytest

from paper_1110_1616_amd import amr as A

CUS, ZCHUNK = 256, 16


def cycle_lists(params, grids):
    arr = (A.amr_grid * len(grids))(*grids)
    out, n = (C.c_int32 * 256)(), C.c_int32()
    fn = A.lib().amr_selfcheck_work_lists
    fn.argtypes = [C.POINTER(A.amr_params), C.c_void_p, C.c_int32, C.c_int32, C.c_void_p, C.POINTER(C.c_int32)]
    assert fn(C.byref(params), arr, len(grids), 64, out, C.byref(n)) == A.AMR_OK
    return [tuple(out[4 * c:4 * c + 4]) for c in range(n.value)]


def columns(n):
    """(tiles, planes) of the flux and the fused list of one grid from band 2:
    predicted states on the grid and one cell around it, updates on the grid
    (and its last z-face)."""
    t = [min(-(-w // (tw - ov)) * -(-h // (256 // tw - ov)) for tw in range(4, 65) if 256 // tw > ov)
         for w, h, ov in ((n[0] + 2, n[1] + 2, 1), (n[0], n[1], 2))]
    return (t[0], n[2] + 2), (t[1], n[2] + 1)


def items(t, d, z):
    return t * -(-d // z)


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("n", [(2, 2, 2), (5, 9, 3), (14, 14, 1), (15, 14, 17), (37, 33, 35), (16, 16, 300), (72, 72, 72)])
def test_short_lists_have_the_shortest_items_with_a_cu_each(n, dtype):
    p = A.make_params(3, n, 1, 2, 4, dtype)
    (flux, flux_long, fused, fused_long), = cycle_lists(p, A.make_grids([(0, (0, 0, 0), n)]))
    for (t, d), got, longest in zip(columns(n), (flux, fused), (flux_long, fused_long)):
        assert items(t, d, ZCHUNK) < CUS
        # the shortest items of which no more than one a CU are needed
        z = min(z for z in range(1, ZCHUNK + 1) if items(t, d, z) <= CUS)
        assert longest == -(-d // -(-d // z)), (longest, z)
        if d > 1 and t * d <= CUS:
            assert longest == 1
        assert got >= items(t, d, z) and (got > items(t, d, ZCHUNK) or d == 1 or z == ZCHUNK)
        if longest <= 8:  # (no item long enough to have its tail cut)
            assert got == items(t, d, z) <= CUS


@pytest.mark.parametrize("n", [(160, 160, 160), (128, 128, 128), (240, 200, 33)])
def test_long_lists_keep_the_configured_items(n):
    p = A.make_params(3, n, 1, 2, 4, "f32")
    (flux, flux_long, fused, fused_long), = cycle_lists(p, A.make_grids([(0, (0, 0, 0), n)]))
    (t, d), (tx, dx) = columns(n)
    assert items(t, d, ZCHUNK) >= CUS and items(tx, dx, ZCHUNK) >= CUS
    assert flux == items(t, d, ZCHUNK) and flux_long == -(-d // -(-d // ZCHUNK))
    # the fused list's shortest items, the last 8% of the work (an item's planes
    # and three more), are cut to at most 8 planes, its others kept
    c = -(-dx // ZCHUNK)
    lengths = sorted(((dx * (i + 1) // c - dx * i // c) for i in range(c) for _ in range(tx)), reverse=True)
    total, acc, want = sum(v + 3 for v in lengths), 0, 0
    for v in lengths:
        acc += v + 3
        want += -(-v // 8) if acc * 100 > total * 92 and v > 8 else 1
    assert fused == want and fused_long == lengths[0]


def test_every_cycle_of_a_hierarchy_is_counted():
    from paper_1110_1616_amd import inputs as I
    grids = I.amr_hierarchy(3, (24, 24, 24), 3, seed=11, ext=(8, 16))
    p = A.make_params(3, (24, 24, 24), 3, 2, 4)
    lists = cycle_lists(p, A.make_grids(grids))
    assert len(lists) == 4
    for flux, flux_long, fused, fused_long in lists:
        assert flux > 0 and fused > 0 and 1 <= flux_long <= ZCHUNK and 1 <= fused_long <= ZCHUNK
