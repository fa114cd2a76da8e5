"""CG on trilinear elements with p . Ap reduced by the operator, in each of its three kernels and in
orders with one and several elements per block (last blocks ragged): the reported residual of a
solve to 1e-10 is the oracle's true residual to 1e-12 of the right-hand side (FP64 rounding over a
few dozen iterations), and it converges in the iterations of the same solve with the separate
summation pass, within one (the reductions are grouped differently)."""
import numpy as np
import pytest
import torch

import workload as wl
from oracle.sem import SemBox
from paper_2210_03179_amd.solver import SemSolver

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("variant", ["0", "1", "2"])
@pytest.mark.parametrize("N", [2, 3, 4, 5, 7, 9])
def test_trilinear_krylov(N, variant, monkeypatch):
    print(f"trilinear CG order {N} variant {variant}", flush=True)
    V = wl.deformed_box((5, 3, 4), 0.04)
    box = SemBox(V, N)
    b = box.mass() * wl.manufactured_load(box.coords())
    monkeypatch.setenv("SEMCHEB_AX_VARIANT", variant)
    kw = dict(N=N, smoother="cheb4", pre=2, post=2, krylov="pcg", geometry="trilinear")
    u, info = SemSolver(V, **kw).solve(torch.from_numpy(b).cuda(), rtol=1e-10, maxit=100)
    nb = np.linalg.norm(b)
    true = np.linalg.norm(b - box.apply(u.cpu().numpy())) / nb
    assert info.relres <= 1e-10 and abs(true - info.relres) <= 1e-12
    monkeypatch.setenv("SEMCHEB_FUSED_KRYLOV", "0")
    _, apart = SemSolver(V, **kw).solve(torch.from_numpy(b).cuda(), rtol=1e-10, maxit=100)
    assert abs(apart.iterations - info.iterations) <= 1
