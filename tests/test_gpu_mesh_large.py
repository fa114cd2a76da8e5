"""Meshes of more than 2,097,152 unknowns, where a Chebyshev step takes two unknowns per thread: 11^3
elements of order 12 (131^3 unknowns, not a multiple of the 512 of a block) against the same box
through the box path, unknowns matched by position. FP64 cycles to 1e-12, mixed cycles (the same BF16
factors, FP32 sums in another order) to 2^-9 of the largest value, node by node."""
import numpy as np
import pytest
import torch
from scipy.spatial import cKDTree

import workload as wl
from paper_2210_03179_amd.solver import MeshSolver, SemSolver

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("smoother", ["cheb4", "cheb1"])
def test_large_mesh_cycles(smoother):
    V = wl.deformed_box((11, 11, 11), 0.05)
    xyz, ev = wl.box_as_mesh(V)
    idx = None
    for precision in ("fp64", "mixed"):
        print(f"large mesh {smoother} {precision}", flush=True)
        kw = dict(N=12, precision=precision, lambda_max=[2.5] * 2, smoother=smoother, pre=3, post=2)
        sb, sm = SemSolver(V, **kw), MeshSolver(xyz, ev, **kw)
        assert sm.n == 131 ** 3 and sm.n > 2048 * 1024
        if idx is None:
            d, idx = cKDTree(sb.coords().cpu().numpy()).query(sm.coords().cpu().numpy())
            assert d.max() < 1e-12
        r = wl.uniform_noise(sb.n, 2)
        zb = sb.vcycle(torch.from_numpy(r).cuda()).cpu().numpy()[idx]
        zm = sm.vcycle(torch.from_numpy(r[idx]).cuda()).cpu().numpy()
        if precision == "fp64":
            assert np.linalg.norm(zm - zb) <= 1e-12 * np.linalg.norm(zb)
        else:
            assert np.max(np.abs(zm - zb)) <= 2.0 ** -9 * np.max(np.abs(zb))
        sb.close(), sm.close()
