"""Nested-dissection steps of 4096 row groups or more, which run one wavefront per group instead of
four: 30 x 34 x 28 elements, with FP64 factors and with their single-precision copies. One cycle of a
one-level order-1 hierarchy inverts the assembled operator to 1e-11 (the factors' rounding times the
condition number, below 3e4), and the mixed cycle stays within 1e-5 of the one with FP64 factors (the
bounds of the smaller boxes)."""
import numpy as np
import pytest
import torch

import workload as wl
from oracle.sem import SemBox
from paper_2210_03179_amd.solver import SemSolver

pytestmark = pytest.mark.gpu
M = (30, 34, 28)


def many_groups(s):
    groups = s.host_array("coarse_steps").reshape(-1, 2)[:, 0]
    return groups.max() >= 4096 > groups.min()


def test_many_groups_invert():
    print(f"dissection steps of {M}", flush=True)
    V = wl.deformed_box(M, 0.05)
    box = SemBox(V, 1)
    s = SemSolver(V, N=1, orders=[1])
    assert many_groups(s)
    r = wl.uniform_noise(box.n, 7)
    z = s.vcycle(torch.from_numpy(r).cuda()).cpu().numpy()
    assert np.linalg.norm(box.apply(z) - r) <= 1e-11 * np.linalg.norm(r)


def test_many_groups_single_precision_factors():
    print(f"dissection steps of {M}, single-precision factors", flush=True)
    V = wl.deformed_box(M, 0.05)
    kw = dict(N=2, orders=[2, 1], lambda_max=[2.5], precision="mixed")
    z = []
    for storage in ("fp64", "mixed"):
        s = SemSolver(V, coarse_storage=storage, **kw)
        assert many_groups(s)
        z.append(s.vcycle(torch.from_numpy(wl.uniform_noise(s.n, 8)).cuda()).cpu().numpy())
    assert np.linalg.norm(z[0] - z[1]) <= 1e-5 * np.linalg.norm(z[0])
