"""Schwarz smoothing at the orders the parity tests leave out (one to four wavefronts per
extended element, even and odd line lengths): one V-cycle against the oracle's definition
(oracle/schwarz.py) with the same lambda_max on both sides. Tolerance: 1e-12 as for the other
orders, scaled by the growth of the operator's rounding with the order, ((N+1)/6)^2 from N = 5."""
import numpy as np
import pytest
import torch

import workload as wl
from oracle import chebyshev as cheb
from oracle import mg
from paper_2210_03179_amd.solver import SemSolver

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sw", ["asm", "ras"])
@pytest.mark.parametrize("N", [3, 4, 6, 8, 9, 12])
def test_schwarz_cycle_orders(N, sw):
    print(f"schwarz {sw} N={N}", flush=True)
    V = wl.deformed_box((3, 2, 2), 0.05)
    lmax = [2.0]  # a bound above the spectrum is not needed for one cycle
    ref = mg.sem_hierarchy(V, N, cheb.CHEB4, 2, 1, orders=[N, 1], lmax=lmax, schwarz=sw)
    s = SemSolver(V, N=N, orders=[N, 1], smoother="cheb4", pre=2, post=1, lambda_max=lmax, schwarz=sw)
    r = wl.uniform_noise(ref.levels[0].n, 22)
    z, zo = s.vcycle(torch.from_numpy(r).cuda()).cpu().numpy(), ref.vcycle(r)
    assert np.linalg.norm(z - zo) <= 1e-12 * max(1.0, ((N + 1) / 6) ** 2) * np.linalg.norm(zo)
