"""GPU: completion flags of the serving loop.  A request that fills the HBM
budget holds the next ones back, so that they are admitted as one batch."""
import time

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_0901_0638_amd as qm  # noqa: E402


@pytest.fixture
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def wait(ctx, tickets, seconds=60):
    end = time.time() + seconds
    while any(qm.qm_poll(ctx, t) == qm.QM_PENDING for t in tickets):
        assert time.time() < end, "not complete"
    assert all(qm.qm_poll(ctx, t) == qm.QM_OK for t in tickets)


def quantile(x, y):
    return qm.make_request(qm.QM_NORMAL_QUANTILE, x, y)


def submit_group(ctx, x, y, smalls):
    """Tickets of a request of the whole budget, then of `smalls` (outputs, in
    order) and one request of the rest of the budget, admitted together."""
    used = sum(s.numel() for s in smalls)
    reqs = [quantile(x, y[0])] + [quantile(x[:s.numel()], s) for s in smalls] + [quantile(x[used:], y[1][used:])]
    tickets = [qm.qm_submit(ctx, r) for r in reqs]     # well within the first one's time
    return tickets[0], tickets[1:-1], tickets[-1]


def test_flags_do_not_wait_for_the_callers_streams(gpu):
    """The first flagged batch of a context completes while the caller's
    default stream is busy: the serving streams are not ordered after it."""
    n = 1 << 25
    x = torch.rand(n, device="cuda", dtype=torch.float64).clamp_(1e-6, 1 - 1e-6)
    y = [torch.empty_like(x) for _ in range(2)]
    smalls = [torch.zeros(4096, device="cuda", dtype=torch.float64) for _ in range(8)]
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    torch.cuda._sleep(1000)
    ev[0].record()
    torch.cuda._sleep(1000000)
    ev[1].record()
    torch.cuda.synchronize()
    half_second = int(1000000 * 500 / ev[0].elapsed_time(ev[1]))
    ctx = qm.Context(0, hbm_budget_bytes=16 * n)
    try:
        # the scheduler, the kernel's code and the staging memory of uploaded batches
        wait(ctx, [qm.qm_submit(ctx, quantile(x[:4096], smalls[0]))])
        for _ in range(6):
            qm.qm_run_batch(ctx, [quantile(x[:1024], y[0][1024 * i:1024 * (i + 1)]) for i in range(20)]
                            + [quantile(x, y[1])], device_tensor=x)
        torch.cuda.synchronize()

        def busy():
            torch.cuda._sleep(half_second)
            e = torch.cuda.Event()
            e.record()
            return e

        e = busy()
        wait(ctx, [qm.qm_submit(ctx, quantile(x, y[0]))])
        shared = e.query()
        torch.cuda.synchronize()
        if shared:
            pytest.skip("the serving and the default stream share a hardware queue")
        e = busy()
        block, small, big = submit_group(ctx, x, y, smalls)
        wait(ctx, [block, *small, big])
        assert not e.query(), "the batch waited for the default stream"
        torch.cuda.synchronize()
        want = torch.empty_like(x)
        qm.qm_normal_quantile(ctx, x, want)
        assert all(torch.equal(s, want[:4096]) for s in smalls)
        used = 8 * 4096
        assert torch.equal(y[0], want) and torch.equal(y[1][used:], want[used:])
    finally:
        ctx.close()


@pytest.mark.parametrize("total,sizes", [
    ((1 << 24) - (1 << 16), [4096] * 8),
    (1 << 26, [1 << 15] * 40),
    (1 << 26, [1, 8192, 8193, 50001, 1 << 17]),       # 1, 1, 2, 7 and 16 chunks of 8192
])
def test_small_requests_complete_before_their_batch(gpu, total, sizes):
    """Small requests beside a large one, however few elements the batch has
    and however late they are in it: each is seen complete before the large one
    (in one of five batches at least: the scheduler may look late), batch after
    batch on the same counts, with its output whole when it is reported."""
    x = torch.rand(total, device="cuda", dtype=torch.float64).clamp_(1e-6, 1 - 1e-6)
    want = torch.empty_like(x)
    y = [torch.empty_like(x) for _ in range(2)]
    smalls = [torch.zeros(n, device="cuda", dtype=torch.float64) for n in sizes]
    used = sum(sizes)
    ctx = qm.Context(0, hbm_budget_bytes=16 * total)
    try:
        qm.qm_normal_quantile(ctx, x, want)
        torch.cuda.synchronize()
        early = [0] * len(sizes)
        for turn in range(6):
            for s in smalls:
                s.zero_()
            torch.cuda.synchronize()
            block, small, big = submit_group(ctx, x, y, smalls)
            for s, t in zip(smalls, small):
                wait(ctx, [t])
                assert torch.equal(s, want[:s.numel()])
            wait(ctx, [block, big])
            end = qm.qm_poll_times(ctx, big)[2]
            if turn:
                early = [e + (qm.qm_poll_times(ctx, t)[2] < end) for e, t in zip(early, small)]
            assert torch.equal(y[1][used:], want[used:])
        assert min(early) > 0, early
    finally:
        ctx.close()


def test_staging_is_made_before_traffic(gpu):
    """The serving loop has its staging slots when the first request is
    admitted, and makes none while batches that need them run."""
    total = 1 << 24
    x = torch.rand(total, device="cuda", dtype=torch.float64).clamp_(1e-6, 1 - 1e-6)
    y = [torch.empty_like(x) for _ in range(2)]
    smalls = [torch.zeros(4096, device="cuda", dtype=torch.float64) for _ in range(40)]
    ctx = qm.Context(0, hbm_budget_bytes=16 * total)
    try:
        slots = lambda: qm.load().qm_debug_staging_slots(ctx.handle)  # noqa: E731
        assert slots() == 0
        wait(ctx, [qm.qm_submit(ctx, quantile(x[:4096], smalls[0]))])
        made = slots()
        assert made >= 4
        for _ in range(6):
            block, small, big = submit_group(ctx, x, y, smalls)
            wait(ctx, [block, *small, big])
        assert slots() == made
    finally:
        ctx.close()
