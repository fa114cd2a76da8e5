"""Which levels setup times on evicted data: those that fit the last-level cache although an iteration
on the finest level does not. In a mixed context an iteration streams the FP64 Krylov operator beside
the single-precision ones, so 24^3 elements of order 7 (113 MB single precision, 396 MB FP64) evict
their single-precision levels. No GPU: the rule is host code of the library."""
import ctypes as C

import pytest

from paper_2210_03179_amd import _lib as L


@pytest.mark.parametrize("level,finest,fp64,mixed,trilinear,cold", [
    ((24, 7), (24, 7), False, True, False, True),     # evicted by the FP64 operator alone
    ((24, 3), (24, 7), False, True, False, True),
    ((24, 7), (24, 7), True, True, False, False),     # does not fit: streams from HBM warm or not
    ((24, 3), (24, 7), True, False, False, True),
    ((16, 7), (16, 7), True, False, False, False),    # 117 MB: nothing evicts it
    ((16, 7), (16, 7), False, True, False, False),    # 117 + 34 MB
    ((32, 7), (32, 7), False, True, False, False),    # 268 MB single precision
    ((24, 7), (24, 7), False, True, True, False),     # trilinear: 113 + 57 MB
    ((32, 7), (32, 7), False, True, True, True),      # 134 MB beside 268 MB
])
def test_cold_levels(level, finest, fp64, mixed, trilinear, cold):
    rule = L.load()["_ZN7semcheb13autotune_coldEllbbb"]
    rule.restype, rule.argtypes = C.c_bool, [C.c_int64] * 2 + [C.c_bool] * 3
    nodes = [m ** 3 * (N + 1) ** 3 for m, N in (level, finest)]
    assert rule(*nodes, fp64, mixed, trilinear) == cold
