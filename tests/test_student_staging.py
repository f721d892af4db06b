"""CPU: what a Student t launch stages in LDS."""
import ctypes
import math

import pytest

import paper_0901_0638_amd as qm


def staging(nu, f32):
    y, lds = ctypes.c_double(), ctypes.c_ulonglong()
    rows = qm.load().qm_debug_student_staging(nu, f32, ctypes.byref(y), ctypes.byref(lds))
    return rows, y.value, lds.value


@pytest.mark.parametrize("f32", [0, 1])
def test_identity_stages_nothing(f32):
    """nu = +inf has no cells: no rows, no LDS, no limit."""
    assert staging(math.inf, f32) == (0, 0.0, 0)


@pytest.mark.parametrize("nu", [0.3, 1.0, 2.9, 4.0, 50.0, 1e6])
def test_staged_rows_reach_ten(nu):
    """|z| <= 10 is served from LDS, whatever the inputs' distribution, within
    the LDS a batch may ask for."""
    for f32 in (0, 1):
        rows, y, lds = staging(nu, f32)
        assert rows >= 1 and y >= 100.0 and lds <= 65536 - 8192 - 256, (nu, f32, rows, y, lds)
