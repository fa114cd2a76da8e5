"""The exact order-1 solve on boxes whose tree cuts the long axis first, with few points across: one
cycle of a one-level order-1 hierarchy inverts the assembled operator. The factors' rounding is
amplified by at most the operator's condition number, about 0.4 over the smallest spacing squared,
below 4e4 here: 1e-11 relative, as for the cubes."""
import numpy as np
import pytest
import torch

import workload as wl
from oracle.sem import SemBox
from paper_2210_03179_amd.solver import SemSolver

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [(12, 11, 130), (6, 6, 400), (9, 9, 170)])
def test_long_box_inverts(m):
    print(f"long box {m}", flush=True)
    V = wl.deformed_box(m, 0.02)
    box = SemBox(V, 1)
    assert box.n > 4096
    s = SemSolver(V, N=1, orders=[1])
    assert len(s.host_array("coarse_steps").reshape(-1, 2)) > 3
    r = wl.uniform_noise(box.n, 7)
    z = s.vcycle(torch.from_numpy(r).cuda()).cpu().numpy()
    assert np.linalg.norm(box.apply(z) - r) <= 1e-11 * np.linalg.norm(r)
