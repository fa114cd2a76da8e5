"""Sparse-level cycles (one launch per Chebyshev step, the small levels in one block) against the
oracle's FD hierarchy, one V-cycle each, at the edges of the dispatch: levels just below and above
the 1024 rows of the one-block kernel, a dense last level of one unknown, of 225 and of 961 (too
large for it), restrictions of 9 and of 225 entries per row, every combination of empty, single
and longer smoothings, all four kinds. Same lambda_max on both sides; FP64 sums of at most 225
terms per row over at most 30 products per cycle: 1e-12 relative."""
import numpy as np
import pytest
import torch

import workload as wl
from oracle import fd2d
from oracle.lanczos import lambda_max_SA
from paper_2210_03179_amd.solver import FdSolver

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,factor,coarsest", [(32, 2, 2), (66, 2, 2), (64, 2, 16), (64, 2, 32), (64, 8, 2), (40, 8, 2)])
@pytest.mark.parametrize("kind,pre,post", [("cheb4opt", 4, 0), ("cheb4", 1, 1), ("cheb1", 3, 2), ("cheb1opt", 0, 3),
                                           ("cheb1opt", 2, 5), ("cheb4", 1, 0), ("cheb4opt", 0, 2)])
def test_fd_cycle_parity(n, factor, coarsest, kind, pre, post):
    print(f"fd cycle n={n} by {factor} to {coarsest}, {kind} ({pre},{post})", flush=True)
    As, _, _ = fd2d.hierarchy_matrices(n, factor, 2.0, 1.0, coarsest)
    lmax = [lambda_max_SA(lambda x, A=A: A @ x, 1.0 / A.diagonal(), A.shape[0]) for A in As[:-1]]
    ref = fd2d.fd_hierarchy(n, factor, kind, pre, post, Lx=2.0, coarsest_n=coarsest, lmax=lmax)
    s = FdSolver(n=n, Lx=2.0, factor=factor, coarsest_n=coarsest, smoother=kind, pre=pre, post=post, lambda_max=lmax)
    b = wl.fd_rhs(n - 1, 3)
    s.reset_counts()
    z = s.vcycle(torch.from_numpy(b).cuda()).cpu().numpy()
    zo = ref.vcycle(b)
    assert np.linalg.norm(z - zo) <= 1e-12 * np.linalg.norm(zo)
    assert s.apply_counts()[:-1] == [pre + post] * (s.num_levels - 1)
