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
