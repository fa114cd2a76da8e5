"""Unstructured-mesh kernels at the edges of their dispatch: a vertex of twelve elements (copy lists
past the eight entries read together), order pairs without compiled transfers, and the fused Krylov
reductions against the separate ones. Against the oracle's SemMesh, the tolerances of the other
mesh tests: operator 1e-14 (N+1)^2, FP64 cycles 1e-12, the mixed cycle 2^-9 node by node."""
import numpy as np
import pytest
import torch

import workload as wl
from oracle import chebyshev as cheb, mg
from oracle.mesh import SemMesh
from paper_2210_03179_amd.solver import MeshSolver

pytestmark = pytest.mark.gpu


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float64)).cuda()


def star_mesh(sectors=6, layers=3):
    """A prism over `sectors` quadrilaterals around one axis, `layers` elements high."""
    ang = np.pi * np.arange(2 * sectors) / sectors
    ring = np.stack([np.cos(ang), np.sin(ang)], axis=1) * np.where(np.arange(2 * sectors) % 2, 1.1, 1.0)[:, None]
    plane = np.concatenate([[[0.05, -0.03]], ring])
    nv = len(plane)
    xyz = np.concatenate([np.column_stack([plane, np.full(nv, 0.7 * z)]) for z in range(layers + 1)])
    ev = []
    for z in range(layers):
        for q in range(sectors):
            a, b, c = 1 + 2 * q, 2 + 2 * q, 1 + (2 * q + 2) % (2 * sectors)
            ev.append([z * nv + v for v in (0, a, c, b)] + [(z + 1) * nv + v for v in (0, a, c, b)])
    return xyz, np.array(ev)


@pytest.mark.parametrize("N", [2, 3, 5])
def test_vertex_of_twelve_elements(N):
    print(f"star mesh N={N}", flush=True)
    xyz, ev = star_mesh()
    ref = SemMesh(xyz, ev, N, None)
    s = MeshSolver(xyz, ev, N=N, lambda_max=[2.0] * 3, orders=[N, 1], smoother="cheb4", pre=2, post=1)
    assert s.n == ref.n
    u = wl.uniform_noise(ref.n, 3)
    w, wo = s.apply_A(dev(u)).cpu().numpy(), ref.apply(u)
    assert np.max(np.abs(w - wo)) < 1e-14 * (N + 1) ** 2 * np.max(np.abs(wo))


@pytest.mark.parametrize("orders,pre,post", [([7, 4, 2, 1], 3, 0), ([6, 5, 1], 2, 2), ([7, 3, 1], 0, 2)])
def test_cycle_without_compiled_transfers(orders, pre, post):
    print(f"mesh cycle {orders} ({pre},{post})", flush=True)
    xyz, ev = wl.box_as_mesh(wl.deformed_box((3, 2, 2), 0.06))
    xyz, ev, _ = wl.shuffled_mesh(xyz, ev, 4)
    kw = dict(N=orders[0], orders=orders, smoother="cheb4", pre=pre, post=post, lambda_max=[2.5] * 4)
    s = MeshSolver(xyz, ev, **kw)
    r = wl.uniform_noise(s.n, 9)
    ref = mg.sem_hierarchy((xyz, ev, None), orders[0], cheb.CHEB4, pre, post, orders=orders,
                           lmax=[2.5] * (len(orders) - 1))
    z = s.vcycle(dev(r)).cpu().numpy()
    m = MeshSolver(xyz, ev, precision="mixed", **kw)
    zm = m.vcycle(dev(r)).cpu().numpy()
    zo = ref.vcycle(r)
    assert np.linalg.norm(z - zo) <= 1e-12 * np.linalg.norm(zo)
    assert np.max(np.abs(zm - z)) <= 2.0 ** -7 * np.max(np.abs(z))  # BF16 factors over up to nine products


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("post", [0, 2])
def test_mesh_fused_krylov(precision, post, monkeypatch):
    """p . Ap inside the operator, the residual update over the copy lists and z . r inside the
    prolongation against the separate passes: same iterations, histories within 1e-13 ||b|| (mixed:
    1e-10 ||b||, the FP32 copy of r is rounded from a differently summed r)."""
    print(f"mesh fused Krylov {precision} post={post}", flush=True)
    xyz, ev = wl.box_as_mesh(wl.deformed_box((3, 3, 2), 0.05))
    xyz, ev, _ = wl.shuffled_mesh(xyz, ev, 5)
    hist = []
    for fused in ("1", "0"):
        monkeypatch.setenv("SEMCHEB_FUSED_KRYLOV", fused)
        s = MeshSolver(xyz, ev, N=5, precision=precision, pre=3, post=post, krylov="fcg")
        b = dev(wl.uniform_noise(s.n, 6))
        _, info = s.solve(b, rtol=1e-8)
        hist.append(info.history)
    assert len(hist[0]) == len(hist[1])
    assert np.max(np.abs(hist[0] - hist[1])) <= (1e-13 if precision == "fp64" else 1e-10) * hist[0][0]
