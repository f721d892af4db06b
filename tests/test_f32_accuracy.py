"""CPU: how close the FP32 forms are to the exact value before their rounding,
range by range: no range may be further off than an FP32 seed with one FP64
correction step is there, which is what the stored rationals stand in for."""
import mpmath as mp
import numpy as np

import oracle
from tests.test_coefficients import arrays, exp_refine7


def horner(c, x):
    r = np.zeros_like(x)
    for ck in c:
        r = r * x + ck
    return r


def horner32(c, x):
    """Horner in FP32 with fused steps, on coefficients rounded to FP32."""
    r = np.zeros_like(x)
    for ck in c:
        r = (r.astype(np.float64) * x + float(np.float32(ck))).astype(np.float32)
    return r


def seed(c, v):
    num = (v * horner32(c["QM_SEED_P"], v)).astype(np.float32)
    return (num * (np.float32(1) / horner32(c["QM_SEED_Q"], v))).astype(np.float32).astype(np.float64)


def exact_exp_to_normal(v):
    """Q(v) = Phi^{-1}(1 - e^{-v}/2) as two doubles (to 1e-25 relative)."""
    out = []
    with mp.workdps(30):
        for x in v:
            x = mp.mpf(float(x))
            if x < mp.log(2):
                q = mp.sqrt(2) * mp.erfinv(-mp.expm1(-x))
            else:
                q = mp.findroot(lambda z: mp.log(mp.erfc(z / mp.sqrt(2)) / 2) + x + mp.log(2), mp.sqrt(2 * x))
            out.append((float(q), float(q - mp.mpf(float(q)))))
    return np.array(out).T


def exp9(a):
    """e^a by the degree-9 Taylor polynomial of the reduced argument."""
    k = np.rint(a * 1.4426950408889634074)
    r = (a - k * 0.69314718055994528623) - k * 2.3190468138462996154e-17
    p = np.zeros_like(r)
    for i in range(9, -1, -1):
        p = p * r + 1 / float(mp.factorial(i))
    return np.ldexp(p, k.astype(np.int64))


def no_further_off(x, edges, new, old):
    for lo, hi in zip(edges, edges[1:]):
        at = (x >= lo) & (x < hi)
        assert np.max(np.abs(new[at])) <= np.max(np.abs(old[at])), (lo, hi)


def test_exp_to_normal():
    """Seed v S4/S5 and one Halley step against q(z) = e^{-v}/2."""
    c = arrays()
    v32 = np.unique(np.geomspace(1e-4, 103, 1201).astype(np.float32))
    v = v32.astype(np.float64)
    hi, lo = exact_exp_to_normal(v)
    x0 = seed(c, v32)
    a = (np.longdouble(0.5) * x0 * x0 - v).astype(np.float64)
    t = horner(c["QM_MILLS_P"], x0) / horner(c["QM_MILLS_Q"], x0) - 1.2533141373155002512 * exp9(a)
    old = x0 + t * (1 + 0.5 * x0 * t)
    new = v * horner(c["QM_E32_P"], v) / horner(c["QM_E32_Q"], v)
    no_further_off(v, [1e-4, 1e-3, 1e-2, 0.1, 0.5, 1, 2, 5, 10, 20, 42, 104], (new - hi - lo) / hi, (old - hi - lo) / hi)


def test_outer_quantile():
    """|z| > 1.64: seed v S4/S5 and one Newton step with the Mills ratio."""
    c = arrays()
    p32 = np.unique(np.geomspace(1.4e-45, 0.05, 40001).astype(np.float32))
    p32 = p32[p32 > 0]
    p = p32.astype(np.float64)
    ref = -oracle.norm_quantile(p)
    v32 = (-np.log(2 * p)).astype(np.float32)
    x0 = seed(c, v32)
    tail = p * 2.5066282746310005024 * exp_refine7(0.5 * (x0 * x0))
    old = x0 + (horner(c["QM_MILLS32_P"], x0) / horner(c["QM_MILLS32_Q"], x0) - tail)
    m, e = np.frexp(p)
    v = -(e + 1) * np.log(2.0) - horner(c["QM_D32_LOG"], m - 0.75)
    new = horner(c["QM_D32_OP"], v) / horner(c["QM_D32_OQ"], v)
    no_further_off(ref, [1.64, 1.8, 2, 2.5, 3, 4, 5, 6, 8, 10, 12, 15], new / ref - 1, old / ref - 1)


def test_central_quantile():
    """|u - 1/2| <= 0.45: seed and one Newton step on Phi(z) = u."""
    c = arrays()
    u32 = np.linspace(0.05, 0.95, 100001).astype(np.float32)
    u = u32.astype(np.float64)
    q = u - 0.5
    at = (np.abs(q) <= 0.45) & (q != 0)
    u, q = u[at], q[at]
    ref = oracle.norm_quantile(u)
    qf = q.astype(np.float32)
    rf = (np.float32(0.2025) - qf * qf).astype(np.float32)
    z0 = (qf * horner32(c["QM_C32_SP"], rf) * (np.float32(1) / horner32(c["QM_C32_SQ"], rf))).astype(np.float64)
    y = z0 * z0
    old = z0 - (z0 * horner(c["QM_C32_E"], y) - q) * horner(c["QM_C32_G"], y)
    r = 0.2025 - q * q
    new = q * horner(c["QM_D32_CP"], r) / horner(c["QM_D32_CQ"], r)
    no_further_off(np.abs(q), [0, 0.01, 0.05, 0.1, 0.2, 0.3, 0.35, 0.4, 0.4501], new / ref - 1, old / ref - 1)
