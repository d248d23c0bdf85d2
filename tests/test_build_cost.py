"""What building a hierarchy holds and starts (host only).

Host memory: one level's lists at a time next to the tables that are kept (and a
bounded group of small levels).  On a 6-level tree the lists of every level are
most of the tables once more; with all of them alive at once, and their
concatenations, the peak is far above the tables themselves.

A small single grid's tables (a band of up to 8192 elements) are built on the
caller's thread: the calls do not wait for other threads."""

import resource
import subprocess
import sys

from paper_1110_1616_amd import amr as A

PEAK = """
import resource, sys
sys.path.insert(0, %r)
from paper_1110_1616_amd import amr as A
from paper_1110_1616_amd import inputs as I
grids = A.make_grids(I.amr_hierarchy(3, (100,) * 3, 6, seed=5, ext=(8, 48), log_uniform=True))
p = A.make_params(3, (100,) * 3, 6, 2, 4, "f32")
peak = lambda: resource.getrusage(resource.RUSAGE_SELF).ru_maxrss * 1024
A.amr_validate(A.make_params(2, (8, 8), 1, 2, 4), A.make_grids([(0, (0, 0), (8, 8))]))
base = peak()
st = A.amr_validate(p, grids)
print(peak() - base, 8 * st["copy_entries"] + 16 * st["prolong_entries"])
"""


def test_one_level_of_lists_is_held_at_a_time():
    import os
    root = os.path.dirname(os.path.dirname(os.path.abspath(A.__file__)))
    out = subprocess.run([sys.executable, "-c", PEAK % root], capture_output=True, text=True, check=True)
    grown, tables = (int(v) for v in out.stdout.split())
    print(f"grown by {grown >> 20} MB, tables {tables >> 20} MB")
    assert grown <= 2.0 * tables, (grown, tables)


def test_small_grids_are_built_on_the_calling_thread():
    for n, ghost in (((8, 8), 4), ((32, 32), 4), ((64, 64), 4), ((6, 5, 4), 2)):
        p = A.make_params(len(n), n, 1, 2, ghost)
        grids = A.make_grids([(0, (0,) * len(n), n)])
        A.amr_validate(p, grids)
        before = resource.getrusage(resource.RUSAGE_THREAD).ru_nvcsw
        for _ in range(100):
            A.amr_validate(p, grids)
        waits = resource.getrusage(resource.RUSAGE_THREAD).ru_nvcsw - before
        print(f"{n}: waited {waits} times in 100 calls")
        assert waits < 50
