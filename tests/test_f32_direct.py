"""The FP32+refine forms of the quantile and of exponential -> normal: FP64
rationals rounded once.  CPU: the stored coefficients against the oracle.
GPU: the correctly rounded oracle value, but for the fit's error, at the
edges of the pieces and over their ranges."""
import numpy as np
import pytest

import oracle
from tests.test_coefficients import arrays

# relative errors before the rounding to FP32: the fits' (2.78e-9; 1.83e-9 plus
# the logarithm's 4.54e-9 times phi-to-tail ratio over z, at most 0.3; 9.5e-12)
# with FP64 rounding of the chains on top
TOL_CENTRAL, TOL_OUTER, TOL_EXP = 2.9e-9, 3.4e-9, 1.2e-11


def horner(c, x):
    r = np.zeros_like(x)
    for ck in c:
        r = r * x + ck
    return r


def outer_points():
    p = np.exp(np.linspace(np.log(2.0 ** -149), np.log(0.05), 4001)).astype(np.float32)
    return np.unique(np.concatenate([p, np.float32([0.05, 2.0 ** -149, 2.0 ** -126, 1e-37, 0.03125, 0.015625])]))


@pytest.mark.parametrize("piece", ["central", "outer", "exp"])
def test_coefficients_against_oracle(piece):
    c = arrays()
    if piece == "central":
        q = np.concatenate([np.linspace(-0.45, 0.45, 4001), [1e-8, 1e-3]])
        q = (q + 0.5).astype(np.float32).astype(np.float64) - 0.5
        q = q[(np.abs(q) <= 0.45) & (q != 0)]
        r = 0.2025 - q * q
        got, ref, tol = q * horner(c["QM_D32_CP"], r) / horner(c["QM_D32_CQ"], r), oracle.norm_quantile(q + 0.5), TOL_CENTRAL
    elif piece == "outer":
        p = outer_points().astype(np.float64)
        m, e = np.frexp(p)
        v = -(e + 1) * np.log(2.0) - horner(c["QM_D32_LOG"], m - 0.75)
        got, ref, tol = -horner(c["QM_D32_OP"], v) / horner(c["QM_D32_OQ"], v), oracle.norm_quantile(p), TOL_OUTER
    else:
        v = np.concatenate([np.exp(np.linspace(np.log(1e-30), np.log(103.0), 4001)), [103.0]])
        got, ref, tol = v * horner(c["QM_E32_P"], v) / horner(c["QM_E32_Q"], v), oracle.exp_to_normal(v), TOL_EXP
    assert np.max(np.abs(got / ref - 1)) < tol


@pytest.mark.gpu
@pytest.mark.parametrize("piece", ["central", "outer", "exp"])
def test_device_rounds_the_oracle_value(piece):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_0901_0638_amd as qm
    edge = np.float32([0.05, 0.95])
    for _ in range(4):
        edge = np.concatenate([edge, np.nextafter(edge, np.float32(0)), np.nextafter(edge, np.float32(1))])
    if piece == "central":
        x = np.concatenate([np.linspace(0.05, 0.95, 100001).astype(np.float32), edge, np.float32([0.5, 0.5 + 2 ** -24])])
        tol = TOL_OUTER       # the edges' neighbours are outer elements
    elif piece == "outer":
        p = outer_points()
        x = np.concatenate([p, 1 - p, edge])
        x = x[(x > 0) & (x < 1)]
        tol = TOL_OUTER
    else:
        x = np.exp(np.linspace(np.log(1e-44), np.log(200.0), 100001)).astype(np.float32)
        x = np.concatenate([x, -x, np.float32([103.0, np.nextafter(np.float32(103), np.float32(200)), 0.0])])
        tol = TOL_EXP
    ctx = qm.Context(0)
    try:
        d = torch.from_numpy(x).cuda()
        out = torch.empty_like(d)
        (qm.qm_recycle_exp_to_normal(ctx, d, out) if piece == "exp" else qm.qm_normal_quantile(ctx, d, out, qm.QM_F32_REFINE))
        got = out.cpu().numpy()
    finally:
        ctx.close()
    ref = (oracle.exp_to_normal if piece == "exp" else oracle.norm_quantile)(x.astype(np.float64))
    half_ulp = 0.5 * np.spacing(np.maximum(np.abs(ref).astype(np.float32), np.abs(got))).astype(np.float64)
    err = np.abs(got.astype(np.float64) - ref) - half_ulp - tol * np.abs(ref)
    assert np.all(err <= 0), (x[np.argmax(err)], err.max())
