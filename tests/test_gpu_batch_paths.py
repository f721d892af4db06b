"""GPU: the two ways a batch's descriptors reach the kernel (its arguments, or
an upload), the split into chunks, and the completion counts' reuse.  Outputs
are bitwise those of the single calls."""
import time

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_0901_0638_amd as qm  # noqa: E402

KINDS = (  # kind, dtype, mode, extra arguments of the request
    (qm.QM_NORMAL_QUANTILE, torch.float64, qm.QM_PLAIN, {}),
    (qm.QM_NORMAL_QUANTILE, torch.float32, qm.QM_F32_REFINE, {}),
    (qm.QM_STUDENT_T, torch.float64, qm.QM_PLAIN, {"nu": 4.0}),
    (qm.QM_STUDENT_T, torch.float64, qm.QM_PLAIN, {"nu": 1.0}),
    (qm.QM_STUDENT_T, torch.float32, qm.QM_F32_REFINE, {"nu": 30.0}),
    (qm.QM_EXP_TO_NORMAL, torch.float64, qm.QM_PLAIN, {}),
    (qm.QM_EXP_TO_HYPERBOLIC, torch.float64, qm.QM_PLAIN, {"hyperbolic": (1.0, 0.5, 1.0), "mu": 0.25}),
    (qm.QM_EXP_TO_HYPERBOLIC, torch.float32, qm.QM_F32_REFINE, {"hyperbolic": (1.0, 0.5, 1.0), "mu": 0.25}),
    (qm.QM_EXP_TO_VG, torch.float64, qm.QM_PLAIN, {"nu": 4.25, "hyperbolic": (1.0, 0.3, 0.0)}),
)
SIZES = (1, 2047, 2048, 2049, 5, 16384, 40961, 0, 100003)


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = qm.Context(0, 8 << 30)
    yield c
    c.close()


def single(ctx, kind, x, y, mode, extra):
    if kind == qm.QM_NORMAL_QUANTILE:
        qm.qm_normal_quantile(ctx, x, y, mode)
    elif kind == qm.QM_STUDENT_T:
        qm.qm_recycle_student_t(ctx, x, y, extra["nu"])
    elif kind == qm.QM_EXP_TO_NORMAL:
        qm.qm_recycle_exp_to_normal(ctx, x, y)
    elif kind == qm.QM_EXP_TO_HYPERBOLIC:
        qm.qm_recycle_exp_to_hyperbolic(ctx, x, y, *extra["hyperbolic"], mu=extra["mu"])
    else:
        qm.qm_recycle_exp_to_vg(ctx, x, y, extra["nu"], *extra["hyperbolic"][:2])


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("count,big", [(1, 0), (2, 0), (16, 0), (17, 0), (70, 0), (16, 1 << 26), (3, (1 << 24) + 5)])
def test_descriptors_in_arguments_or_uploaded(ctx, count, big, noalloc):
    """Up to and beyond 16 requests, with and without more chunks than an
    argument batch takes: the single calls' bits, and nothing past the end."""
    g = torch.Generator(device="cuda").manual_seed(count + big)
    reqs, want, got = [], [], []
    for i in range(count):
        kind, dtype, mode, extra = KINDS[i % len(KINDS)]
        n = big if big and i == 0 else SIZES[(i + i // len(SIZES)) % len(SIZES)]
        x = torch.rand(n, generator=g, device="cuda", dtype=dtype).clamp_(1e-6, 1 - 1e-6)
        buf = torch.zeros(n + 1, device="cuda", dtype=dtype)
        y = torch.empty(n, device="cuda", dtype=dtype)
        single(ctx, kind, x, y, mode, extra)
        reqs.append(qm.make_request(kind, x, buf[:n], mode=mode, **extra))
        want.append((x, y))
        got.append(buf)
    run = qm.qm_run_batch_noalloc if noalloc else qm.qm_run_batch
    run(ctx, reqs, device_tensor=got[0])
    torch.cuda.synchronize()
    for i, ((_, y), buf) in enumerate(zip(want, got)):
        assert torch.equal(buf[:-1], y) and buf[-1] == 0, (i, reqs[i].kind, reqs[i].n)


def test_completion_counts_serve_batch_after_batch(ctx):
    """Batches of a large request and small flagged ones, several in a row on
    the same staging: every request completes, with the single call's bits."""
    x = torch.rand(1 << 26, device="cuda", dtype=torch.float64).clamp_(1e-6, 1 - 1e-6)
    want = torch.empty_like(x)
    qm.qm_normal_quantile(ctx, x, want)
    for turn in range(6):
        y = torch.zeros_like(x)
        small = [torch.zeros(n, device="cuda", dtype=torch.float64) for n in (1, 4096, 16384, 70001, 300000)]
        torch.cuda.synchronize()
        reqs = [qm.make_request(qm.QM_NORMAL_QUANTILE, x[:s.numel()], s) for s in small]
        reqs.insert(turn % 6, qm.make_request(qm.QM_NORMAL_QUANTILE, x, y))
        tickets = [qm.qm_submit(ctx, r) for r in reqs]
        end = time.time() + 60
        while any(qm.qm_poll(ctx, t) != qm.QM_OK for t in tickets):
            assert time.time() < end
        assert torch.equal(y, want)
        for s in small:
            assert torch.equal(s, want[:s.numel()])
