"""GMRES vector kernels over long bases: a weak cycle (one step of the 1st kind, coarsening by 8,
stretched grid) needs more than 16 basis vectors, with restarts at 32 (every chunk size of the
projections), 17 and 5; odd and even vector lengths, an iterate that is only 8-byte aligned, and a
capped run whose last queued cycle must not be counted. Against the oracle's GMRES, the tolerances
of the other GMRES tests: identical iterations, recurrences to 1e-11 ||b||, solutions to 1e-10."""
import numpy as np
import pytest
import torch

import workload as wl
from oracle import fd2d, krylov
from oracle.lanczos import lambda_max_SA
from paper_2210_03179_amd.solver import FdSolver

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,restart,maxit", [(32, 32, 200), (32, 17, 200), (33, 32, 200), (32, 5, 200), (32, 32, 9)])
def test_gmres_long_basis(n, restart, maxit):
    print(f"gmres basis n={n} restart={restart}", flush=True)
    f = 8 if n % 8 == 0 else 11
    As, _, _ = fd2d.hierarchy_matrices(n, f, 8.0, 1.0, 2)
    lmax = [lambda_max_SA(lambda x, A=A: A @ x, 1.0 / A.diagonal(), A.shape[0]) for A in As[:-1]]
    if f == 11:  # the library coarsens by 2, 4 or 8: one level, solved exactly, odd-sized
        s = FdSolver(n=n, Lx=8.0, factor=2, coarsest_n=2, smoother="cheb1", pre=1, post=0, krylov="gmres",
                     restart=restart)
        A = As[0]
        ref = lambda r: np.linalg.solve(A.toarray(), r)  # noqa: E731
    else:
        ref = fd2d.fd_hierarchy(n, f, "cheb1", 1, 0, Lx=8.0, coarsest_n=2, lmax=lmax).vcycle
        A = As[0]
        s = FdSolver(n=n, Lx=8.0, factor=f, coarsest_n=2, smoother="cheb1", pre=1, post=0, krylov="gmres",
                     lambda_max=lmax, restart=restart)
    b = wl.fd_rhs(n - 1, 5)
    res = krylov.fgmres(lambda x: A @ x, b, ref, 1e-9, restart=restart, maxit=maxit)
    out = torch.empty(b.size + 1, dtype=torch.float64, device="cuda")[1:]
    s.reset_counts()
    u, info = s.solve(torch.from_numpy(b).cuda(), rtol=1e-9, maxit=maxit, out=out)
    assert u.data_ptr() % 16 == 8 and info.iterations == res.iterations and info.converged == res.converged
    if f == 8 and restart == 32 and maxit == 200:
        assert info.iterations > 16
    h = np.array(res.history)
    assert np.max(np.abs(info.history - h)) <= 1e-11 * np.linalg.norm(b)
    assert np.linalg.norm(u.cpu().numpy() - res.x) <= 1e-10 * np.linalg.norm(res.x)
    restarts = (info.iterations - 1) // restart
    assert s.apply_counts()[0] == info.iterations * (2 if f == 8 else 1) + restarts
