"""Order transfers in both block lengths of their dispatch (standard runs of elements from 256 blocks
on, short runs below): one V-cycle against the oracle on a box whose runs are ragged along x, FP64
to 1e-12, and the mixed cycle within one BF16 unit roundoff per application (2^-7 of the largest
entry over the cycle's products)."""
import numpy as np
import pytest
import torch

import workload as wl
from oracle import chebyshev as cheb, mg
from paper_2210_03179_amd.solver import SemSolver

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [(9, 17, 17), (5, 3, 2)])
@pytest.mark.parametrize("orders", [[4, 2, 1], [5, 3, 1], [6, 3, 1], [3, 1]])
def test_transfer_block_lengths(orders, m):
    print(f"transfers {orders} on {m}", flush=True)
    V = wl.deformed_box(m, 0.04)
    lmax = [2.5] * (len(orders) - 1)
    ref = mg.sem_hierarchy(V, orders[0], cheb.CHEB4, 1, 1, orders=orders, lmax=lmax)
    kw = dict(N=orders[0], orders=orders, smoother="cheb4", pre=1, post=1, lambda_max=lmax)
    r = wl.uniform_noise(ref.levels[0].n, 12)
    zo = ref.vcycle(r)
    z = SemSolver(V, **kw).vcycle(torch.from_numpy(r).cuda()).cpu().numpy()
    assert np.linalg.norm(z - zo) <= 1e-12 * np.linalg.norm(zo)
    zm = SemSolver(V, precision="mixed", **kw).vcycle(torch.from_numpy(r).cuda()).cpu().numpy()
    assert np.max(np.abs(zm - zo)) <= 2.0 ** -7 * np.max(np.abs(zo))
