"""CPU: the power a^rho of the variance-gamma origin series, in the kernels'
steps, against mpmath."""
import ctypes

import mpmath as mp
import numpy as np
import pytest

import paper_0901_0638_amd as qm

# roundings of the reduced exponent (two of 2.8e-17), of the polynomial's last
# step (1.1e-16) and of the one before it (0.35 of 1.6e-16), remainder 4e-18
TOL = 3e-16


@pytest.mark.parametrize("rho", [1.1, 1.5, 4.0 / 3.0, 2.000001, 7.5, 14.8])
def test_power_is_within_an_ulp_or_so(rho):
    rng = np.random.default_rng(5)
    a = np.concatenate([np.exp(-rng.uniform(0, 690 / rho, 1500)), 2.0 ** -rng.integers(0, int(990 / rho), 40),
                        np.sqrt(0.5) * 2.0 ** -np.arange(0, 9), np.nextafter(np.sqrt(0.5) * 2.0 ** -np.arange(0, 9), 0),
                        [1.0, np.nextafter(1.0, 0)]])
    w = np.empty_like(a)
    dp = ctypes.POINTER(ctypes.c_double)
    assert qm.load().qm_debug_pow_small(a.ctypes.data_as(dp), rho, w.ctypes.data_as(dp), a.size) == 0
    with mp.workdps(40):
        err = [abs(float(mp.mpf(float(y)) / mp.power(mp.mpf(float(x)), mp.mpf(rho)) - 1)) for x, y in zip(a, w)]
    assert max(err) <= TOL, (a[int(np.argmax(err))], max(err))


def test_power_of_the_ends():
    a = np.array([0.0, 5e-324, 1e-310, 1e-300])
    w = np.empty_like(a)
    dp = ctypes.POINTER(ctypes.c_double)
    qm.load().qm_debug_pow_small(a.ctypes.data_as(dp), 1.1, w.ctypes.data_as(dp), a.size)
    assert np.isfinite(w[0]) and np.array_equal(w[1:], np.zeros(3))
