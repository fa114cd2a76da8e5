"""Register budgets of the FP64 operator on trilinear elements, read from the metadata of the built
library: the sums of p . Ap ride only in the kernels that store them. A plain application's plane
loop keeps the waves its order leaves it (four up to order 7, three above: 512 registers per lane and
SIMD). Spills: at most a dozen registers with the sums (pencils of order 9, plane loop of order 12),
and plain pencils from order 11 on, which setup times against the plane loop before taking them. No
GPU: the code objects are in the library."""
import glob
import os
import re
import subprocess

import pytest

from paper_2210_03179_amd import _lib as L


def kernels(tmp_path):
    tool = next(iter(glob.glob("/opt/rocm/llvm/bin/llvm-readelf")), None)
    if tool is None:
        pytest.skip("no llvm-readelf in this image")
    blob = open(L.LIB_PATH, "rb").read()
    out = {}
    for m in re.finditer(b"\x7fELF\x02", blob):
        if blob[m.start() + 18:m.start() + 20] != b"\xe0\x00":  # e_machine: AMD GPU
            continue
        part = os.path.join(tmp_path, "part.co")
        with open(part, "wb") as f:
            f.write(blob[m.start():])
        notes = subprocess.run([tool, "--notes", part], capture_output=True, text=True).stdout
        for name, vgprs, spill in re.findall(
                r"\.name:\s+(\S+)\n.*?\.vgpr_count:\s+(\d+)\s+\.vgpr_spill_count:\s+(\d+)", notes, re.S):
            out[name] = (int(vgprs), int(spill))
    return out


def test_trilinear_operator_registers(tmp_path):
    ks = {}
    for name, regs in kernels(str(tmp_path)).items():
        m = re.search(r"ax_tri_kernelILi(\d+)EdLi(\d+)ELi(\d)ELb(\d)E", name)
        if m:
            ks[tuple(int(v) for v in m.groups())] = regs
    assert {k[0] for k in ks} == set(range(1, 13))
    for (order, _, tile, dot), (vgprs, spill) in ks.items():
        if tile == 0 and not dot:
            assert vgprs <= (128 if order <= 7 else 168), (order, vgprs)
        if tile == 1 and dot:
            assert order < 10
        if spill and not (tile == 1 and not dot and order >= 11):
            assert spill <= 12 and (order, tile, dot) in ((9, 1, 1), (12, 0, 1)), (order, tile, dot, spill)
