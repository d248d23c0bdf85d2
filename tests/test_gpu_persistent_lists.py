"""Fused launches from the work queue: lists of more claims than the device holds
blocks (the others run one block a claim), against the two kernels, bit for bit
and over several launches, as each leaves the queue ready for the next."""

import pytest
import torch

from gpu_util import log
from paper_1110_1616_amd import amr as A
from paper_1110_1616_amd import inputs as I

pytestmark = pytest.mark.gpu


# 2-D: 14 x 14 cells an item, 3-D: that times at most zchunk planes; a device of
# 256 CUs holds 512 blocks in FP64, up to 1536 in FP32.  (300, 300) and
# (30, 20, 24): one block a claim, but for claims of one in the largest lists
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n,zchunk", [((300, 300), 16), ((700, 650), 16), ((30, 20, 24), 16), ((100, 90, 130), 2)])
def test_queue_and_block_launches_agree(n, zchunk, dtype):
    nd = len(n)
    ic = I.smooth_mhd(nd, n, seed=13, jump=True)
    H = A.Hierarchy(nd, n, [(0, (0,) * nd, n)], ghost=4, dtype=dtype, dx0=ic["dx"])

    def run(mode):
        log(f"case: {n} {dtype} launch mode {mode}")
        H.set_launch_config(1, zchunk, mode)
        U, V = H.new_state(), H.new_state()
        H.load_primitive(U, 0, ic["prim"], ic["b"])
        for s in range(6):
            if s % 2 == 0:
                H.fill(0, A.AMR_FILL_SAME_LEVEL, U)
            H.compute_dt(U)
            H.advance(U, V, cycle=0, band=4 - 2 * (s % 2))
            U, V = V, U
        assert H.error_flags()[0] == 0
        return H.store_interior(U, 0)

    want = run(0)
    for mode in (8, 10, 9, 12, 14, 12 | 16, 14 | 16, 12 | 48):
        for f, a, b in zip(A.FIELDS, run(mode), want):
            assert (a == b).all(), (mode, f)
    torch.cuda.synchronize()
