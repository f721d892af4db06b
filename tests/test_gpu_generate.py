"""GPU parity: fused generation (qm_generate).  The device's Philox4x32-10
and the host generator (qm_inputs) are independent implementations of the
published definition, so the uniforms must agree bit for bit; the mapped
outputs must be bitwise those of qm_normal_quantile on the host's uniforms,
and within tolerance of the oracle."""
import ctypes
import math

import numpy as np
import pytest

import oracle
import qm_inputs as qi
from tests._tol import RTOL_F32, RTOL_F64, as_f32_output, assert_close

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_0901_0638_amd as qm  # noqa: E402


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = qm.Context(0)
    yield c
    c.close()


def gen(ctx, seed, stream, first, n, dtype, kind, mode=None, offset=0):
    """Generate into out[offset:offset+n] of a fresh zeroed buffer (offset
    shifts the output's alignment); returns the whole buffer."""
    t = torch.zeros(n + offset + 1, dtype=dtype, device="cuda")
    qm.qm_generate(ctx, seed, stream, first, t[offset:offset + n], kind, mode)
    torch.cuda.synchronize()
    return t.cpu().numpy()


@pytest.mark.parametrize("seed,stream", [(0, 0), (1, 7), (0xFFFFFFFF, 0xFFFFFFFF), (12345, 1000)])
def test_uniforms_bitwise_equal_host_generator(ctx, seed, stream):
    for dtype, host in ((torch.float64, qi.uniform53), (torch.float32, qi.uniform23)):
        n = 100003
        got = gen(ctx, seed, stream, 0, n, dtype, qm.QM_UNIFORM)[:n]
        ref = host(seed, stream, n)
        assert np.array_equal(got, ref), (dtype, seed, stream, np.flatnonzero(got != ref)[:5])
        assert got.min() > 0 and got.max() < 1


@pytest.mark.parametrize("first", [0, 1, 2, 3, 5, 1 << 33, (1 << 40) + 7])
@pytest.mark.parametrize("offset", [0, 1, 3])
def test_uniform_subranges_and_alignment(ctx, first, offset):
    """Any sub-range, at any output alignment: equal to the host's elements
    first .. first+n-1 (regenerated by index on the host), and nothing
    written outside the range."""
    n = 4099
    for dtype, host in ((torch.float64, qi.uniform53), (torch.float32, qi.uniform23)):
        buf = gen(ctx, 3, 9, first, n, dtype, qm.QM_UNIFORM, offset=offset)
        if first < (1 << 20):
            ref = host(3, 9, first + n)[first:]
        else:
            ref = host_range(host, 3, 9, first, n, dtype)
        assert np.array_equal(buf[offset:offset + n], ref), (dtype, first, offset)
        assert np.all(buf[:offset] == 0) and buf[offset + n] == 0


def host_range(host, seed, stream, first, n, dtype):
    """Elements first .. first+n-1 of a host stream far from its start, from
    single Philox blocks (the host generator's block function)."""
    out = np.empty(n, np.float64 if dtype == torch.float64 else np.float32)
    per = 2 if dtype == torch.float64 else 4
    key = np.array([seed, stream], np.uint32)
    for i in range(n):
        e = first + i
        b = e // per
        w = qi.philox4x32_10(np.array([b & 0xFFFFFFFF, b >> 32, 0, 0], np.uint32), key)
        if per == 2:
            lo, hi = (w[0], w[1]) if e % 2 == 0 else (w[2], w[3])
            out[i] = qi.u53_of_bits([(int(hi) << 32) | int(lo)])[0]
        else:
            out[i] = qi.u23_of_words([int(w[e % 4])])[0]
    return out


def test_device_philox_known_answer(ctx):
    """Block 0 of key (0, 0) is the published all-zero known-answer vector
    of Philox4x32-10 (SC'11): the device's first uniforms are the open-uniform
    formulas of those words."""
    words = [0x6627E8D5, 0xE169C58D, 0xBC57AC4C, 0x9B00DBD8]
    want64 = qi.u53_of_bits([(words[1] << 32) | words[0], (words[3] << 32) | words[2]])
    want32 = qi.u23_of_words(words)
    got64 = gen(ctx, 0, 0, 0, 2, torch.float64, qm.QM_UNIFORM)[:2]
    got32 = gen(ctx, 0, 0, 0, 4, torch.float32, qm.QM_UNIFORM)[:4]
    assert np.array_equal(got64, want64) and np.array_equal(got32, want32)


@pytest.mark.parametrize("dtype,mode,rtol", [(torch.float64, qm.QM_PLAIN, RTOL_F64), (torch.float64, qm.QM_PAPER, RTOL_F64),
                                             (torch.float32, qm.QM_F32_REFINE, RTOL_F32),
                                             (torch.float32, qm.QM_PLAIN, RTOL_F32),
                                             (torch.float32, qm.QM_PAPER, 5e-7)])
def test_fused_quantile_equals_two_step_and_oracle(ctx, dtype, mode, rtol):
    """Fused Phi^{-1} of the stream = qm_normal_quantile of the host's
    uniforms, bitwise, at several offsets and alignments; and the oracle's
    w(u) within the form's tolerance (the paper's FP32 (5,6) is good to 5e-7
    on its domain, which open 24-bit uniforms never leave)."""
    host = qi.uniform53 if dtype == torch.float64 else qi.uniform23
    for first, offset, n in ((0, 0, 1 << 18), (1, 0, 7777), (2, 1, 5000), (3, 3, 129), (0, 0, 1), (5, 0, 3)):
        u = host(11, 4, first + n)[first:]
        fused = gen(ctx, 11, 4, first, n, dtype, qm.QM_NORMAL_QUANTILE, mode, offset)[offset:offset + n]
        d = torch.from_numpy(u).cuda()
        w = torch.empty_like(d)
        qm.qm_normal_quantile(ctx, d, w, mode)
        torch.cuda.synchronize()
        two = w.cpu().numpy()
        assert np.array_equal(fused, two), (mode, first, offset, n)
        assert_close(fused, oracle.norm_quantile(u.astype(np.float64)), rtol, "fused %s %d" % (mode, first))


def test_fused_full_size_sampled(ctx):
    """2^28 FP64 samples in one launch (the benchmark's shape): sampled
    outputs against the oracle at host-regenerated uniforms."""
    n = 1 << 28
    t = torch.empty(n, dtype=torch.float64, device="cuda")
    qm.qm_generate(ctx, 0, 0, 0, t, qm.QM_NORMAL_QUANTILE)
    torch.cuda.synchronize()
    rng = np.random.default_rng(5)
    idx = np.unique(np.concatenate([rng.integers(0, n, 1 << 12), [0, 1, n - 2, n - 1]]))
    got = t[torch.from_numpy(idx).cuda()].cpu().numpy()
    uu = np.array([host_range(qi.uniform53, 0, 0, int(i), 1, torch.float64)[0] for i in idx])
    assert_close(got, oracle.norm_quantile(uu), RTOL_F64, "fused 2^28 sampled")


def test_generate_errors(ctx):
    lib = qm.load()
    d = torch.zeros(8, dtype=torch.float64, device="cuda")
    p = ctypes.c_void_p(d.data_ptr())
    assert lib.qm_generate(ctx.handle, 1 << 32, 0, 0, p, 8, qm.QM_UNIFORM, qm.QM_F64, qm.QM_PLAIN, None) == qm.QM_E_INVAL
    assert lib.qm_generate(ctx.handle, 0, 1 << 32, 0, p, 8, qm.QM_UNIFORM, qm.QM_F64, qm.QM_PLAIN, None) == qm.QM_E_INVAL
    assert lib.qm_generate(ctx.handle, 0, 0, 1 << 63, p, 8, qm.QM_UNIFORM, qm.QM_F64, qm.QM_PLAIN, None) == qm.QM_E_INVAL
    assert lib.qm_generate(ctx.handle, 0, 0, 0, p, 8, qm.QM_STUDENT_T, qm.QM_F64, qm.QM_PLAIN, None) == qm.QM_E_INVAL
    assert lib.qm_generate(ctx.handle, 0, 0, 0, p, 8, qm.QM_UNIFORM, qm.QM_F64, qm.QM_PAPER, None) == qm.QM_E_DTYPE
    assert lib.qm_generate(ctx.handle, 0, 0, 0, p, 8, qm.QM_NORMAL_QUANTILE, qm.QM_F64, qm.QM_F32_REFINE,
                           None) == qm.QM_E_DTYPE
    assert lib.qm_generate(ctx.handle, 0, 0, 0, None, 8, qm.QM_UNIFORM, qm.QM_F64, qm.QM_PLAIN, None) == qm.QM_E_INVAL
    assert lib.qm_generate(ctx.handle, 0, 0, 0, ctypes.c_void_p(d.data_ptr() + 4), 2, qm.QM_UNIFORM, qm.QM_F64,
                           qm.QM_PLAIN, None) == qm.QM_E_INVAL
    assert lib.qm_generate(ctx.handle, 0, 0, 0, None, 0, qm.QM_UNIFORM, qm.QM_F64, qm.QM_PLAIN, None) == qm.QM_OK
    # a failed call leaves the output untouched
    torch.cuda.synchronize()
    assert np.all(d.cpu().numpy() == 0)


def gen_student(ctx, seed, stream, first, n, dtype, nu, offset=0):
    t = torch.zeros(n + offset + 1, dtype=dtype, device="cuda")
    qm.qm_generate_student_t(ctx, seed, stream, first, t[offset:offset + n], nu)
    torch.cuda.synchronize()
    return t.cpu().numpy()


@pytest.mark.parametrize("nu", [0.5, 1.0, 4.0, 30.0, 1e6, float("inf")])
def test_fused_student_t_equals_two_call_chain(ctx, nu):
    """Fused uniform -> normal -> Student t: bitwise the recycling map of the
    normals qm_generate writes (FP64 and FP32+refine), at several stream
    offsets and output alignments, and within tolerance of the oracle's map
    of those same normals."""
    rng = np.random.default_rng(int(min(nu, 1e6) * 10))
    for dtype in (torch.float64, torch.float32):
        for first, offset, n in ((0, 0, 70001), (3, 1, 4099), (1 << 33, 3, 2049)):
            got = gen_student(ctx, 11, 5, first, n, dtype, nu, offset)[offset:offset + n]
            z = torch.from_numpy(gen(ctx, 11, 5, first, n, dtype, qm.QM_NORMAL_QUANTILE)[:n]).cuda()
            t = torch.empty_like(z)
            qm.qm_recycle_student_t(ctx, z, t, nu)
            torch.cuda.synchronize()
            ref = t.cpu().numpy()
            assert np.array_equal(got.view(np.uint8), ref.view(np.uint8)), (nu, dtype, first, offset)
            if np.isfinite(nu) and first == 0:
                idx = np.unique(rng.integers(0, n, 300))
                zs = z.cpu().numpy()[idx].astype(np.float64)
                want = oracle.student_t_map(zs, nu)
                rtol = RTOL_F64 if dtype == torch.float64 else RTOL_F32
                assert_close(got[idx], as_f32_output(want) if dtype == torch.float32 else want, rtol, "nu=%s" % nu)


def host_base(u, lp, lm, alpha, beta):
    """The two-sided exponential base sample of qm_generate_hyperbolic, in numpy FP64.
    p+- come from the C library's exp, as the library forms them: near
    u = p-, v is ill-conditioned in p- itself (a last-bit difference in p-
    moves v by ~1/|u - p-| ulps), so the reference must use the same p-."""
    u = np.asarray(u, np.float64)
    pm, pp = math.exp(lm), math.exp(lp)
    inv_m, inv_p = 1.0 / (alpha + beta), 1.0 / (alpha - beta)
    neg = u < pm
    ratio = np.where(neg, u * (1.0 / pm), (1.0 - u) * (1.0 / pp))
    return np.log(ratio) * np.where(neg, inv_m, -inv_p)


@pytest.mark.parametrize("p", [(1.0, 0.0, 1.0), (1.0, 0.5, 1.0), (2.0, -1.5, 0.3)], ids=lambda p: "a%g_b%g_d%g" % p)
def test_fused_hyperbolic(ctx, p):
    """Fused uniform -> base sample -> hyperbolic: against the oracle's map
    of the base samples formed on the host from the device's own uniforms
    (the host and device logarithms may differ by an ulp, which the map
    passes on at most about one to one)."""
    lp, lm = qm.qm_hyperbolic_masses(ctx, *p)
    rng = np.random.default_rng(5)
    for dtype in (torch.float64, torch.float32):
        for first, offset, n in ((0, 0, 50001), (5, 1, 4099)):
            t = torch.zeros(n + offset + 1, dtype=dtype, device="cuda")
            qm.qm_generate_hyperbolic(ctx, 21, 2, first, t[offset:offset + n], *p, mu=0.0)
            torch.cuda.synchronize()
            got = t.cpu().numpy()[offset:offset + n]
            assert t.cpu().numpy()[offset + n] == 0, "wrote past the range"
            u = gen(ctx, 21, 2, first, n, dtype, qm.QM_UNIFORM)[:n]
            v = host_base(u, lp, lm, p[0], p[1])
            idx = np.unique(np.concatenate([rng.integers(0, n, 400), [np.argmax(v), np.argmin(v)]]))
            want = oracle.hyperbolic_map(v[idx], *p)
            if dtype == torch.float64:
                assert_close(got[idx], want, RTOL_F64, "fused hyperbolic %r" % (p,))
            else:
                assert_close(got[idx], as_f32_output(want), RTOL_F32, "fused hyperbolic f32 %r" % (p,))
            assert np.array_equal(np.sign(got), np.sign(v))


def test_fused_chains_reject_bad_arguments(ctx):
    out = torch.zeros(16, dtype=torch.float64, device="cuda")
    with pytest.raises(qm.QMError):
        qm.qm_generate_student_t(ctx, 1, 0, 0, out, 0.1)
    with pytest.raises(qm.QMError):
        qm.qm_generate_student_t(ctx, 1 << 32, 0, 0, out, 4.0)
    with pytest.raises(qm.QMError):
        qm.qm_generate_hyperbolic(ctx, 1, 0, 0, out, 1.0, 1.0, 1.0)
    with pytest.raises(qm.QMError):
        qm.qm_generate_hyperbolic(ctx, 1, 0, 0, out, 1.0, 0.0, 1.0, mode=qm.QM_PAPER)


@pytest.mark.parametrize("p", [(2, 1.0, 0.5), (3, 2.0, -1.0)], ids=lambda p: "l%d_a%g_b%g" % p)
def test_fused_vg(ctx, p):
    """Fused uniform -> base sample -> variance-gamma, checked like the
    hyperbolic chain."""
    lp, lm = qm.qm_vg_masses(ctx, *p)
    rng = np.random.default_rng(9)
    for dtype in (torch.float64, torch.float32):
        n = 30001
        t = torch.zeros(n, dtype=dtype, device="cuda")
        qm.qm_generate_vg(ctx, 31, 4, 0, t, *p)
        torch.cuda.synchronize()
        got = t.cpu().numpy()
        u = gen(ctx, 31, 4, 0, n, dtype, qm.QM_UNIFORM)[:n]
        v = host_base(u, lp, lm, p[1], p[2])
        idx = np.unique(rng.integers(0, n, 400))
        want = oracle.vg_map(v[idx], *p)
        if dtype == torch.float64:
            assert_close(got[idx], want, RTOL_F64, "fused vg %r" % (p,))
        else:
            assert_close(got[idx], as_f32_output(want), RTOL_F32, "fused vg f32 %r" % (p,))


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("first", [1, 2, 3])
@pytest.mark.parametrize("n", [2, 63, 511, 514, 1 << 12, (1 << 14) + 5])
def test_fused_chains_at_any_block_offset_and_alignment(ctx, dtype, first, n):
    """Ranges that start inside a Philox block, written at every offset from a
    16-byte boundary, around the sizes of a wave's tile: bitwise the same
    elements of an aligned run from the stream's start, and nothing outside."""
    runs = (lambda f, out: qm.qm_generate_student_t(ctx, 21, 6, f, out, 4.0),
            lambda f, out: qm.qm_generate_hyperbolic(ctx, 21, 6, f, out, 1.0, 0.5, 1.0, mu=0.25))
    for run in runs:
        whole = torch.empty(first + n, dtype=dtype, device="cuda")
        run(0, whole)
        for offset in range(16 // whole.element_size()):
            t = torch.zeros(n + offset + 1, dtype=dtype, device="cuda")
            run(first, t[offset:offset + n])
            torch.cuda.synchronize()
            assert torch.equal(t[offset:offset + n], whole[first:]), (first, offset, n)
            assert torch.all(t[:offset] == 0) and t[offset + n] == 0
