"""What contexts keep on the device. hipMalloc hands out memory in pieces of up to 2 MB, so the bounds
leave 10 % of the arrays in question."""
import torch
import pytest

import workload as wl
from paper_2210_03179_amd.solver import BatchedSolver, SemSolver

pytestmark = pytest.mark.gpu


def used_by(make):
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    s = make()
    used = free - torch.cuda.mem_get_info()[0]
    s.close()
    return used


def test_ras_keeps_own_nodes_only():
    """RAS holds (N+1)^3 results per element in both precisions where ASM holds (N+3)^3."""
    print("memory of RAS and ASM", flush=True)
    V = wl.deformed_box((20, 20, 20), 0.05)
    kw = dict(N=7, precision="mixed", lambda_max=[2.0] * 2, orders=[7, 1])
    used_by(lambda: SemSolver(V, schwarz="ras", **kw))  # device libraries and pools in place
    asm = used_by(lambda: SemSolver(V, schwarz="asm", **kw))
    ras = used_by(lambda: SemSolver(V, schwarz="ras", **kw))
    assert asm - ras >= 0.9 * 8000 * (10 ** 3 - 8 ** 3) * 12


def test_batch_keeps_no_single_solver_vectors():
    """Batched solves have no z and no A p: two FP64 vectors less per system than its single solver."""
    print("memory of a batch", flush=True)
    verts = [wl.deformed_box((10, 10, 10), 0.05) for _ in range(6)]
    single = [used_by(lambda V=V: SemSolver(V, N=7, precision="mixed")) for V in verts + verts[:1]][1:]
    batch = [used_by(lambda: BatchedSolver(verts, [7] * 6)) for _ in range(2)][1]  # the first loads its kernels
    assert sum(single) - batch >= 0.9 * 6 * 2 * 8 * 69 ** 3 - 2 ** 22
