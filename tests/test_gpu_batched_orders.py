"""Every order a batch takes (4..12) in one batch, on boxes whose element runs are ragged along x:
the transfers and operators of all orders share launches there. Each solution meets the solve's
1e-8 in the true FP64 residual of the oracle's operator, the reported residual is that residual
(1e-10 of the right-hand side: FP64 rounding over a few dozen iterations), and the system's own
single-system solve converges alike: within one iteration, and with both residuals below 1e-8 |b|
the difference d of the two solutions has |A d| <= 2.02e-8 |b|."""
import numpy as np
import pytest
import torch

import workload as wl
from oracle.sem import SemBox
from paper_2210_03179_amd import _lib as L
from paper_2210_03179_amd.solver import BatchedSolver, SemSolver

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pre,post,krylov", [(2, 2, "pcg"), (3, 0, "fcg"), (2, 2, "fcg")])
@pytest.mark.parametrize("orders", [list(range(4, 13)), [6], [12, 4, 4]])
def test_batched_orders(orders, pre, post, krylov):
    print(f"batch of orders {orders} ({pre},{post}) {krylov}", flush=True)
    verts = [wl.batched_box(2 + q % 4, 900 + q) for q in range(len(orders))]
    boxes = [SemBox(V, N) for V, N in zip(verts, orders)]
    rhs = [bx.mass() * wl.manufactured_load(bx.coords()) for bx in boxes]
    kw = dict(smoother="cheb4", pre=pre, post=post, krylov=krylov)
    bs = BatchedSolver(verts, orders, **kw)
    u, st, its, rel = bs.solve(torch.from_numpy(np.concatenate(rhs)).cuda(), rtol=1e-8, maxit=300)
    assert st == L.SEM_OK
    uh = u.cpu().numpy()
    for q, (V, N, bx, bq) in enumerate(zip(verts, orders, boxes, rhs)):
        uq = uh[bs.offsets[q]:bs.offsets[q + 1]]
        nb = np.linalg.norm(bq)
        res = np.linalg.norm(bq - bx.apply(uq))
        assert res <= 1.01e-8 * nb, (q, N, res / nb)
        assert abs(res / nb - rel[q]) <= 1e-10, (q, N)
        us, info = SemSolver(V, N=N, precision="mixed", **kw).solve(torch.from_numpy(bq).cuda(), rtol=1e-8,
                                                                    maxit=300)
        assert abs(info.iterations - its[q]) <= 1, (q, N)
        d = us.cpu().numpy() - uq
        assert np.linalg.norm(bx.apply(d)) <= 2.02e-8 * nb, (q, N)
