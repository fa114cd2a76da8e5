"""The one-thread-per-pencil operator (FP64 variants 3 and 5, BF16 variant 4, trilinear variant
2) at the orders the variant tests leave out: odd and even N + 1 (the even-odd products have a
middle row and column for even N), orders whose element spans several waves, element counts that
do not fill a block. FP64 against the oracle to 1e-14 (N+1)^2, the bound of the other variants
(90 rounding units times (N+1)^2); BF16 factors against the plane loop with the same factors
(variant 0) to the same 90 units times (N+1)^2 in single precision."""
import numpy as np
import pytest
import torch

import workload as wl
from oracle.sem import SemBox
from paper_2210_03179_amd.solver import SemSolver

pytestmark = pytest.mark.gpu


def relmax(a, b):
    return np.max(np.abs(a - b)) / np.max(np.abs(b))


@pytest.mark.parametrize("N", [1, 2, 6, 8, 10, 11, 12])
def test_pencil_operator_orders(N, monkeypatch):
    print(f"pencil operator N={N}", flush=True)
    V = wl.deformed_box((3, 3, 2), 0.06)
    box = SemBox(V, N)
    u = wl.uniform_noise(box.n, 31)
    ref = box.apply_local(box.scatter(u)).ravel()
    ut = torch.from_numpy(u).cuda()
    out32 = {}
    for v in (0, 3, 4, 5):
        monkeypatch.setenv("SEMCHEB_AX_VARIANT", str(v))
        s = SemSolver(V, N=N, lambda_max=[1.0] * 8, orders=[N, 1] if N > 1 else [1], precision="mixed")
        assert relmax(s.apply_local(ut).cpu().numpy(), ref) < 1e-14 * (N + 1) ** 2, v
        if N > 1:
            out32[v] = s.apply_local(ut.float()).double().cpu().numpy()
        s.close()
    if N > 1:  # a one-level hierarchy stores no BF16 factors
        assert relmax(out32[4], out32[0]) < 90 * 2.0 ** -24 * (N + 1) ** 2


@pytest.mark.parametrize("N", [2, 3, 7, 10])
def test_pencil_operator_reduces_p_Ap(N, monkeypatch):
    """The p . Ap partials of the Krylov operator (blocks of several elements, a ragged last
    block): a solve with the reduction inside the operator against the separate summation pass,
    same iterations, residual history within 1e-13 ||b||."""
    print(f"pencil p.Ap N={N}", flush=True)
    V = wl.deformed_box((3, 2, 3), 0.05)
    b = torch.from_numpy(wl.uniform_noise(SemBox(V, N).n, 32)).cuda()
    monkeypatch.setenv("SEMCHEB_AX_VARIANT", "5")
    hist = []
    for fused in ("1", "0"):
        monkeypatch.setenv("SEMCHEB_FUSED_KRYLOV", fused)
        s = SemSolver(V, N=N)
        _, info = s.solve(b, rtol=1e-8)
        hist.append(info.history)
        s.close()
    assert len(hist[0]) == len(hist[1])
    assert np.max(np.abs(hist[0] - hist[1])) <= 1e-13 * hist[0][0]
