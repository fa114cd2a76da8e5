"""The nested-dissection factorisation (boxes of more than 4096 order-1 unknowns) under
AddressSanitizer and UndefinedBehaviorSanitizer, with the build, runtime and checks of the other
sanitizer test: a near-cube of two levels of threads (many small fronts side by side, few large ones
with the threads inside), a long box and one a single point across. No GPU."""
import os
import subprocess
import sys

import pytest

from test_host_sanitizers import ROOT, _runtime

SCRIPT = r"""
import sys
sys.modules["torch"] = None          # host-only: the binding must not need torch here
sys.path.insert(0, ROOT)
import workload as wl
from paper_2210_03179_amd.solver import SemSolver
for m, steps in (((18, 17, 19), 3), ((5, 5, 280), None), ((2, 70, 62), None), ((20, 9, 33), None)):
    s = SemSolver(wl.deformed_box(m, 0.05), N=1, orders=[1], device=-1)
    st = s.host_array("coarse_steps").reshape(-1, 2)
    assert len(st) > 1 and (steps is None or len(st) == steps), (m, len(st))
    s.close()
print("SANITIZED RUN OK")
"""


@pytest.mark.slow
def test_dissection_under_sanitizers(tmp_path):
    asan = _runtime("asan")
    if asan is None:
        pytest.skip("no clang AddressSanitizer runtime in this image")
    from paper_2210_03179_amd.build import build_host_sanitized
    lib = build_host_sanitized(str(tmp_path))
    env = dict(os.environ, SEMCHEB_LIB=lib, LD_PRELOAD=asan,
               ASAN_OPTIONS="detect_leaks=0:halt_on_error=1:abort_on_error=0",
               UBSAN_OPTIONS="halt_on_error=1:print_stacktrace=1", OMP_NUM_THREADS="4")
    r = subprocess.run([sys.executable, "-c", SCRIPT.replace("ROOT", repr(ROOT))], env=env, capture_output=True,
                       text=True, timeout=900)
    report = r.stdout[-3000:] + r.stderr[-6000:]
    assert r.returncode == 0, report
    assert "SANITIZED RUN OK" in r.stdout, report
    assert "AddressSanitizer" not in r.stderr and "runtime error" not in r.stderr, report
