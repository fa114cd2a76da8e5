"""Trilinear elements at the orders between and above those of the other trilinear tests: the plain
application and the one with the p . Ap sums are kernels of their own, and from order 10 on the sums
always ride in the plane loop. CG on every variant against the oracle's operator: the recurrence's
residual is the true one to 1e-12 of the right-hand side, the operator matches to 1e-14 (N+1)^2, and
separate sums change the iteration count by at most one (the bounds of the other trilinear tests)."""
import numpy as np
import pytest
import torch

import workload as wl
from oracle.sem import SemBox
from paper_2210_03179_amd.solver import SemSolver

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("variant", ["0", "1", "2"])
@pytest.mark.parametrize("N", [6, 8, 10, 11, 12])
def test_trilinear_orders(N, variant, monkeypatch):
    print(f"trilinear order {N} variant {variant}", flush=True)
    V = wl.deformed_box((3, 2, 3), 0.04)
    box = SemBox(V, N)
    b = box.mass() * wl.manufactured_load(box.coords())
    monkeypatch.setenv("SEMCHEB_AX_VARIANT", variant)
    kw = dict(N=N, smoother="cheb4", pre=2, post=2, krylov="pcg", geometry="trilinear")
    s = SemSolver(V, **kw)
    x = wl.uniform_noise(box.n, 5)
    w, wo = s.apply_A(torch.from_numpy(x).cuda()).cpu().numpy(), box.apply(x)
    assert np.max(np.abs(w - wo)) <= 1e-14 * (N + 1) ** 2 * np.max(np.abs(wo))
    u, info = s.solve(torch.from_numpy(b).cuda(), rtol=1e-10, maxit=100)
    true = np.linalg.norm(b - box.apply(u.cpu().numpy())) / np.linalg.norm(b)
    assert info.relres <= 1e-10 and abs(true - info.relres) <= 1e-12
    monkeypatch.setenv("SEMCHEB_FUSED_KRYLOV", "0")
    _, apart = SemSolver(V, **kw).solve(torch.from_numpy(b).cuda(), rtol=1e-10, maxit=100)
    assert abs(apart.iterations - info.iterations) <= 1
