"""GPU: the shared tile walk.  Outputs must not depend on where the arrays lie
or on the launch: every (input, output) offset from a 16-byte boundary and
sizes around a lane's vectors, a wave's tile and the vectors-per-lane rule
give, bit for bit, the elements of one aligned launch; elements beyond the
LDS cells may sit anywhere, several to a lane."""
import numpy as np
import pytest

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


MAPS = {
    "quantile": lambda c, x, y: qm.qm_normal_quantile(c, x, y, qm.QM_PLAIN if x.dtype == torch.float64 else qm.QM_F32_REFINE),
    "exp_normal": qm.qm_recycle_exp_to_normal,
    "student": lambda c, x, y: qm.qm_recycle_student_t(c, x, y, 4.0),
    "student_1": lambda c, x, y: qm.qm_recycle_student_t(c, x, y, 1.0),
    "hyperbolic": lambda c, x, y: qm.qm_recycle_exp_to_hyperbolic(c, x, y, 1.0, 0.5, 1.0, mu=0.25),
    "vg_origin": lambda c, x, y: qm.qm_recycle_exp_to_vg(c, x, y, 4.25, 1.0, 0.3, mu=-0.5),
}
TOP = (1 << 19) + 7      # two vectors per lane begin below this in FP64, above it in FP32


def inputs(name, dtype, n):
    rng = np.random.default_rng(17)
    if name == "quantile":
        x = rng.random(n)
        x[rng.random(n) < 0.1] = 1e-30
        special = [0.0, 1.0, 0.5, np.nan, -1.0, 2.0]
    else:
        x = rng.standard_normal(n) * rng.choice([1e-6, 0.01, 1.0, 3.0, 30.0], n)
        special = [0.0, -0.0, np.inf, -np.inf, np.nan, 1e300, -700.0, 5e-324]
    at = rng.permutation(n)[:len(special) * 8]
    x[at] = np.resize(special, at.size)
    with np.errstate(over="ignore"):
        return torch.from_numpy(x).to(dtype).cuda()


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("name", sorted(MAPS))
def test_any_offset_and_size_equals_one_aligned_launch(ctx, name, dtype):
    run = MAPS[name]
    x = inputs(name, dtype, TOP)
    want = torch.empty_like(x)
    run(ctx, x, want)
    per = 16 // x.element_size()
    for n in (1, per - 1, per, per + 1, 64 * per - 1, 64 * per + 1, 256 * per + 3, 4099, TOP - 2 * per):
        for i in range(per):
            for o in range(per):
                xi = torch.empty(n + per, dtype=dtype, device="cuda")[i:i + n]
                xi.copy_(x[per:per + n])
                buf = torch.zeros(n + per + 1, dtype=dtype, device="cuda")
                run(ctx, xi, buf[o:o + n])
                a, b = buf[o:o + n], want[per:per + n]
                assert torch.equal(torch.nan_to_num(a, nan=123.0), torch.nan_to_num(b, nan=123.0)), (name, n, i, o)
                assert torch.all(buf[:o] == 0) and torch.all(buf[o + n:] == 0), (name, n, i, o)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("name", ["student", "student_1", "hyperbolic", "vg_origin"])
def test_far_elements_anywhere_equal_a_launch_of_their_own(ctx, name, dtype):
    """Waves of far elements only, and one far element at every position of a
    lane's eight: the same bits as that element mapped alone."""
    run = MAPS[name]
    far = torch.tensor([11.0, -38.0, 200.0, -1e-7, 1e-5, 0.0, 900.0, -20.5], dtype=dtype, device="cuda")
    alone = torch.empty_like(far)
    for k in range(far.numel()):
        run(ctx, far[k:k + 1], alone[k:k + 1])
    x = far.repeat(1 << 14)
    y = torch.empty_like(x)
    run(ctx, x, y)
    assert torch.equal(y, alone.repeat(1 << 14))
    near = torch.full((1 << 17,), 0.75, dtype=dtype, device="cuda")
    base = torch.empty_like(near)
    run(ctx, near, base)
    at = torch.arange(0, near.numel(), 37, device="cuda")
    near[at] = far[at % 8]
    run(ctx, near, y[:near.numel()])
    base[at] = alone[at % 8]
    assert torch.equal(y[:near.numel()], base)


BIG = {"quantile": (25, 26), "exp_normal": (25, 26), "student": (24, 24), "student_1": (24, 24), "hyperbolic": (24, 24),
       "vg_origin": (24, 24)}      # log2 of the vectors (FP64, FP32) from which a workgroup takes two tiles


@pytest.mark.parametrize("huge", [False, True])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("name", sorted(BIG))
def test_large_launches_equal_small_ones(ctx, name, dtype, huge):
    """From the first size on with two tiles to a workgroup, and from that
    with one of four vectors: an even and an odd number of tiles, whole and
    with a partial last one, element by element the values of a small launch."""
    x = inputs(name, dtype, TOP)
    want = torch.empty_like(x)
    MAPS[name](ctx, x, want)
    per = 16 // x.element_size()
    first = per << (27 if huge else BIG[name][dtype == torch.float32])
    n = first + 1024 * per + 5
    reps = -(-n // TOP)
    xs = x.repeat(reps)[:n]
    as_int = torch.int64 if dtype == torch.float64 else torch.int32
    want = torch.where(torch.isnan(want), torch.full_like(want, float("nan")), want).view(as_int)
    for m in (first, first + 1024 * per, n):
        y = torch.full((n,), 7.0, dtype=dtype, device="cuda")
        MAPS[name](ctx, xs[:m], y[:m])
        assert bool((y[m:] == 7.0).all())
        whole = m // TOP * TOP
        y.masked_fill_(torch.isnan(y), float("nan"))
        got = y.view(as_int)
        assert bool((got[:whole].view(-1, TOP) == want).all()), (name, m)
        assert bool((got[whole:m] == want[:m - whole]).all()), (name, m)
        del y, got
