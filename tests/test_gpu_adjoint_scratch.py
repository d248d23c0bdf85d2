"""The reverse steps' scratch arrays give their place to later ones, and a
segment's step states are replicated from its checkpoint: neither may let what
the workspace held before, or how a run is cut into segments, into the
result.  Both are exact (the same operations on the same values), so the
tolerance is zero."""

import numpy as np
import pytest

from paper_1110_1616_amd import inputs as I

pytestmark = pytest.mark.gpu


def _grids(ndim, n, tiles):
    if tiles == 1:
        return [((0,) * ndim, n)]
    h = n[0] // 2
    return [((0,) * ndim, (h,) + n[1:]), ((h,) + (0,) * (ndim - 1), n)]


@pytest.mark.parametrize("ndim,n,tiles,dtype", [
    (2, (9, 8), 1, "f32"), (2, (67, 31), 2, "f64"),
    (3, (8, 9, 8), 1, "f64"), (3, (21, 10, 13), 2, "f32"),
])
@pytest.mark.parametrize("nsteps", [1, 4])
def test_adjoint_reads_nothing_stale(ndim, n, tiles, dtype, nsteps):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1110_1616_amd import amr as A
    ic = I.smooth_mhd(ndim, n, seed=4, v_rms=0.1, b_rms=0.3, p_amp=0.1)
    boxes = _grids(ndim, n, tiles)
    H = A.Hierarchy(ndim, n, [(0, lo, hi) for lo, hi in boxes], ghost=2, dtype=dtype, dx0=ic["dx"],
                    gamma=5.0 / 3.0)
    dts = [2e-3 + 1e-4 * k for k in range(nsteps)]
    U = H.new_state()
    for gi, f in enumerate(I.split_grid_fields(ic, boxes)):
        H.load_primitive(U, gi, f["prim"], f["b"])
    # the states before each step (forward, one step at a time)
    states, V = [], A.State([f.clone() for f in U.fields])
    for dt in dts:
        states.append(A.State([f.clone() for f in U.fields]))
        H.fill(0, A.AMR_FILL_SAME_LEVEL, U)
        H.dt0.fill_(dt)
        A.amr_advance_patches(H.h, 0, None, 2, U.c, V.c, 0, H.dt0, H.ws)
        U, V = V, U
    rng = np.random.default_rng(8)
    seed = [torch.zeros(H.state_elems, dtype=U.fields[0].dtype, device="cuda") for _ in range(8)]
    for gi in range(len(boxes)):
        A.amr_store_interior_adjoint(
            H.h, gi, [torch.tensor(rng.normal(size=s), device="cuda") for s in H.interior_shapes(gi)],
            A.State(seed).c)

    def reverse(cuts, byte):
        lam = A.State([f.clone() for f in seed])
        ws = torch.full((A.amr_adjoint_workspace(H.h, -1, nsteps),), byte, dtype=torch.uint8, device="cuda")
        for k0, k1 in reversed(cuts):
            A.amr_advance_adjoint(H.h, -1, dts[k0:k1], states[k0].c, lam.c, ws)
        return [H.store_interior(lam, gi) for gi in range(len(boxes))]

    want = reverse([(0, nsteps)], 0)
    assert all(np.isfinite(x).all() for g in want for x in g)
    for cuts, byte in [([(0, nsteps)], 255), ([(k, k + 1) for k in range(nsteps)], 255)]:
        for g, w in zip(reverse(cuts, byte), want):
            for x, y in zip(g, w):
                assert np.array_equal(x, y)
