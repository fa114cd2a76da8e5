"""Meshes with many elements around one vertex: the copies past the eighth go to a list of their own,
and what the lists cost grows with the copies, not with the unknowns times the largest number of
copies. Stars of 3, 4, 7, 8 and 20 sectors and 3 layers: axis vertices of 6, 8 (the slots exactly
full), 14, 16 and 40 elements, axis edges of 3 to 20. Operator against the oracle's SemMesh to 1e-14
(N+1)^2, the FP64 cycle to 1e-12, the mixed solve to its own 1e-8."""
import numpy as np
import pytest
import torch

import workload as wl
from oracle import chebyshev as cheb, mg
from oracle.mesh import SemMesh
from paper_2210_03179_amd.solver import MeshSolver
from test_gpu_mesh_lists import dev, star_mesh

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sectors", [3, 4, 7, 8, 20])
@pytest.mark.parametrize("N", [2, 5])
def test_star_operator_and_cycle(N, sectors):
    print(f"star of {sectors} sectors N={N}", flush=True)
    xyz, ev = star_mesh(sectors=sectors)
    ref = SemMesh(xyz, ev, N, None)
    kw = dict(N=N, lambda_max=[2.0] * 3, orders=[N, 1], smoother="cheb4", pre=2, post=1)
    s = MeshSolver(xyz, ev, **kw)
    u = wl.uniform_noise(ref.n, 3)
    w, wo = s.apply_A(dev(u)).cpu().numpy(), ref.apply(u)
    assert np.max(np.abs(w - wo)) < 1e-14 * (N + 1) ** 2 * np.max(np.abs(wo))
    oracle = mg.sem_hierarchy((xyz, ev, None), N, cheb.CHEB4, 2, 1, orders=[N, 1], lmax=[2.0])
    z, zo = s.vcycle(dev(u)).cpu().numpy(), oracle.vcycle(u)
    assert np.linalg.norm(z - zo) <= 1e-12 * np.linalg.norm(zo)
    m = MeshSolver(xyz, ev, N=N, precision="mixed")
    x, info = m.solve(dev(u), rtol=1e-8)
    assert info.relres <= 1e-8
    assert np.linalg.norm(u - ref.apply(x.cpu().numpy())) <= 1.01e-8 * np.linalg.norm(u)


def test_lists_cost_what_the_copies_cost():
    """4000 elements around an axis, 60 thousand unknowns: all arrays of a context of two levels
    (factors, vectors, maps) take under 400 MB; lists padded to the largest valence alone 1 GB."""
    print("valence 4000", flush=True)
    xyz, ev = star_mesh(sectors=2000, layers=2)
    xyz[::len(xyz) // 3, :2] = 0.0  # thin sectors are convex only around a centred axis
    torch.cuda.synchronize()
    free0 = torch.cuda.mem_get_info()[0]
    s = MeshSolver(xyz, ev, N=3, lambda_max=[2.0] * 3)
    used = free0 - torch.cuda.mem_get_info()[0]
    assert s.n > 60_000 and used < 400e6
