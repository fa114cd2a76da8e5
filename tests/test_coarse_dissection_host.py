"""The tree of the nested-dissection coarse solve on boxes that are long along one axis: cutting such
a box along every axis separates it by whole length-wise planes, whose dense blocks grow with the
length squared. The factor keeps to the entries of the z-plane chain it replaces (three dense blocks
per plane) or 80 MB, and boxes near a cube keep the few steps of cutting all axes. No GPU: host-only
contexts factorise too."""
import numpy as np
import pytest

import workload as wl
from paper_2210_03179_amd.solver import SemSolver


def steps_of(m):
    s = SemSolver(wl.deformed_box(m, 0.05), N=1, orders=[1], device=-1)
    st = s.host_array("coarse_steps").reshape(-1, 2)
    s.close()
    return st


@pytest.mark.parametrize("m", [(17, 17, 150), (6, 6, 400), (150, 9, 9), (9, 120, 9)])
def test_long_boxes_keep_small_factors(m):
    nx, ny, nz = (v - 1 for v in m)
    st = steps_of(m)
    assert nx * ny * nz > 4096 and len(st) > 0
    assert st[:, 1].sum() <= max(3 * nz * (nx * ny) ** 2, 1e7)


@pytest.mark.parametrize("m,steps", [((18, 17, 19), 3), ((24, 24, 24), 5)])
def test_cubes_cut_all_axes(m, steps):
    assert len(steps_of(m)) == steps


def test_dense_boxes_have_no_steps():
    assert steps_of((6, 5, 4)).size == 0 and np.prod((5, 4, 3)) <= 4096
