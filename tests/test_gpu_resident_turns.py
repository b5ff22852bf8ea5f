"""Contexts whose solves run in the resident loop share the device by launches:
a long solve of one does not keep another's from the device until it ends.  In
one server the other requests go on beside a launch of the loop."""
import threading
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_1803_03797_amd import cg  # noqa: E402


@pytest.fixture(scope="module")
def torch():
    t = pytest.importorskip("torch")
    if not t.cuda.is_available():
        pytest.fail("no GPU visible")
    return t


def rhs(torch, nx, ny, seed=1):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.rand(ny, nx, generator=g, device="cuda", dtype=torch.float64) * 2 - 1


def served(ctx, b, x, kw):
    t = ctx.cg_submit(cg.make_problem(b, x, b.shape[1], b.shape[0], **kw))
    while True:
        rc, r = ctx.cg_poll(t)
        if rc != cg.CG_PENDING:
            return rc, r
        time.sleep(0.0002)


def solved(ctx, b, x, kw):
    return ctx.solve(b, x, b.shape[1], b.shape[0], **kw)


@pytest.mark.parametrize("how", [solved, served])
def test_short_solves_beside_a_long_one(torch, how):
    """Five short solves are done while another context's solve of some
    tenths of a second goes on."""
    big, small = rhs(torch, 1024, 1024), rhs(torch, 300, 190, 2)
    long_kw = dict(tol=0.0, maxit=60000, variant=0)
    short_kw = dict(tol=0.0, maxit=300)
    with cg.Context(device=0, arena_bytes=1 << 30) as a, \
            cg.Context(device=0, arena_bytes=1 << 30) as c:
        ref = torch.zeros_like(small)
        how(c, small, ref, short_kw)
        xa = torch.zeros_like(big)
        torch.cuda.synchronize()
        rc = []
        th = threading.Thread(target=lambda: rc.append(solved(a, big, xa, long_kw)))
        th.start()
        time.sleep(0.05)
        got = []
        for _ in range(5):
            x = torch.zeros_like(small)
            how(c, small, x, short_kw)
            got.append((x, th.is_alive()))
            print("short solve", how.__name__, got[-1][1], flush=True)
        th.join()
        print("long solve", rc[0][1].iterations, "%.2f s" % rc[0][1].device_seconds, flush=True)
        assert rc[0][1].iterations > 20000
        for x, beside in got:
            np.testing.assert_array_equal(x.cpu().numpy(), ref.cpu().numpy())
            assert beside
        assert "resident_abandoned" not in a.cg_kernel_stats()
        assert "resident_abandoned" not in c.cg_kernel_stats()


def test_small_requests_beside_a_launch(torch):
    """Small requests, one after the other, do not each wait for a whole launch
    of the loop: on average for less than 160 of a large solve's iterations (a
    launch has 256 when nothing else arrives)."""
    big, small = rhs(torch, 1024, 1024), rhs(torch, 12, 12, 2)
    with cg.Context(device=0, arena_bytes=1 << 30) as c:
        xb, x = torch.zeros_like(big), torch.zeros_like(small)
        torch.cuda.synchronize()
        t = c.cg_submit(cg.make_problem(big, xb, 1024, 1024, tol=0.0, maxit=20000))
        n = 0
        while c.cg_poll(t)[0] == cg.CG_PENDING:
            served(c, small, x, dict(tol=0.0, maxit=1))
            n += 1
        print("served", n, c.cg_kernel_stats(), flush=True)
        assert n > 20000 // 160


def test_calls_on_a_context_that_serves(torch):
    """The server's thread lets other callers of its context in between its
    turns: solves (on chip, in the loop, in a batch) are done while a served
    one goes on."""
    big, mid, small = rhs(torch, 700, 700), rhs(torch, 300, 190, 2), rhs(torch, 33, 17, 3)
    kw = dict(tol=0.0, maxit=40)

    def calls(c):
        x, y = torch.zeros_like(mid), torch.zeros_like(small)
        u, v = torch.zeros_like(mid), torch.zeros_like(small)
        solved(c, small, y, kw)
        solved(c, mid, x, kw)
        c.cg_solve_batch([cg.make_problem(mid, u, 300, 190, **kw),
                          cg.make_problem(small, v, 33, 17, **kw)])
        return [t.cpu().numpy() for t in (x, y, u, v)]

    with cg.Context(device=0, arena_bytes=1 << 30, max_slots=8) as c:
        want = calls(c)
        xb = torch.zeros_like(big)
        torch.cuda.synchronize()
        t = c.cg_submit(cg.make_problem(big, xb, 700, 700, tol=0.0, maxit=40000))
        time.sleep(0.01)
        for _ in range(3):
            for a, b in zip(calls(c), want):
                np.testing.assert_array_equal(a, b)
            assert c.cg_poll(t)[0] == cg.CG_PENDING
            print("calls beside a served solve", flush=True)
        while c.cg_poll(t)[0] == cg.CG_PENDING:
            time.sleep(0.001)
        ref = torch.zeros_like(big)
        solved(c, big, ref, dict(tol=0.0, maxit=40000))
        np.testing.assert_array_equal(xb.cpu().numpy(), ref.cpu().numpy())
