"""GMRES vector kernels over long bases at an even vector length (1232 unknowns, whole 16-byte packs):
a weak cycle (one step, lambda_max twice the true one) takes 48 to 63 iterations, so bases of up to 32,
17 and 6 vectors fill and restart; with an iterate that is 16- or only 8-byte aligned. Against the
oracle's GMRES with the tolerances of the other GMRES tests: identical iterations, recurrences to 1e-11
||b||, solutions to 1e-10."""
import numpy as np
import pytest
import torch

import workload as wl
from oracle import chebyshev as cheb, krylov, mg
from oracle.sem import SemBox
from paper_2210_03179_amd.solver import SemSolver

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("restart,offset", [(32, 0), (32, 1), (17, 0), (6, 1)])
def test_gmres_even_length(restart, offset):
    print(f"gmres even length, restart {restart}, offset {offset}", flush=True)
    V = wl.deformed_box((5, 4, 3), 0.05)
    box = SemBox(V, 3)
    assert box.n % 2 == 0
    kw = dict(N=3, orders=[3, 1], smoother="cheb4", pre=1, post=0, lambda_max=[4.0])
    ref = mg.sem_hierarchy(V, 3, cheb.CHEB4, 1, 0, orders=[3, 1], lmax=[4.0])
    b = box.mass() * wl.manufactured_load(box.coords()) + 1e-3 * wl.uniform_noise(box.n, 3)
    res = krylov.fgmres(box.apply, b, ref.vcycle, 1e-9, restart=restart, maxit=120)
    assert res.converged and res.iterations > 32
    s = SemSolver(V, krylov="gmres", restart=restart, **kw)
    out = torch.empty(box.n + 1, dtype=torch.float64, device="cuda")[offset:offset + box.n]
    s.reset_counts()
    u, info = s.solve(torch.from_numpy(b).cuda(), rtol=1e-9, maxit=120, out=out)
    assert u.data_ptr() % 16 == 8 * offset and info.converged and info.iterations == res.iterations
    assert np.max(np.abs(info.history - np.array(res.history))) <= 1e-11 * np.linalg.norm(b)
    assert np.linalg.norm(u.cpu().numpy() - res.x) <= 1e-10 * np.linalg.norm(res.x)
    restarts = (info.iterations - 1) // restart
    assert s.apply_counts()[0] == info.iterations * 2 + restarts
