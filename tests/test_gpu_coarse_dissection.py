"""The exact order-1 solve by nested dissection (boxes of more than 4096 order-1 unknowns): a
one-level hierarchy of order 1 is the coarse solve alone, so one cycle must invert the assembled
operator. Boxes with one and two interior points along an axis, ragged splits, and the same box
through the z-plane blocking. Tolerance on the residual: the factors' rounding is amplified by at
most the condition number of the operator, about 0.4 h^-2 < 3e4 here: 1e-11 relative."""
import numpy as np
import pytest
import torch

import workload as wl
from oracle.sem import SemBox
from paper_2210_03179_amd.solver import SemSolver

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [(18, 17, 19), (2, 80, 70), (61, 3, 46), (40, 25, 6), (24, 24, 24)])
def test_nested_dissection_inverts(m):
    print(f"nested dissection {m}", flush=True)
    V = wl.deformed_box(m, 0.05)
    box = SemBox(V, 1)
    assert box.n > 4096
    s = SemSolver(V, N=1, orders=[1])
    r = wl.uniform_noise(box.n, 7)
    z = s.vcycle(torch.from_numpy(r).cuda()).cpu().numpy()
    assert np.linalg.norm(box.apply(z) - r) <= 1e-11 * np.linalg.norm(r)
    blocked = SemSolver(V, N=1, orders=[1], coarse_planes=1)
    zb = blocked.vcycle(torch.from_numpy(r).cuda()).cpu().numpy()
    assert np.linalg.norm(z - zb) <= 1e-11 * np.linalg.norm(zb)


def test_nested_dissection_single_precision_factors():
    """coarse_storage="mixed": the mixed cycle reads single-precision copies of the factors; the
    cycle stays within 1e-5 of the one with FP64 factors (the bound of the blocked factors' test)."""
    V = wl.deformed_box((18, 17, 19), 0.05)
    kw = dict(N=3, orders=[3, 1], lambda_max=[2.5], precision="mixed")
    z = []
    for storage in ("fp64", "mixed"):
        s = SemSolver(V, coarse_storage=storage, **kw)
        z.append(s.vcycle(torch.from_numpy(wl.uniform_noise(s.n, 8)).cuda()).cpu().numpy())
    assert np.linalg.norm(z[0] - z[1]) <= 1e-5 * np.linalg.norm(z[0])
