"""GPU parity of the on-chip solver at the limits of its forms: 2, 5, 10 or 20
rows a thread, the least that keeps (nx + 1) * ceil(ny / rows) within 512
threads.  Every arithmetic step and the order of every sum are the oracle's, so
iterates are compared bit for bit."""
import sys

import numpy as np
import pytest

import oracle
from oracle import MODE_CANONICAL
from paper_1803_03797_amd import cg

pytestmark = pytest.mark.gpu

# (nx, ny, rows): the last grid of a form and the first of the next, at widths
# on and off the wavefront size, with whole and ragged last segments
SHAPES = [(63, 16, 2), (63, 17, 5), (63, 39, 5), (63, 40, 5), (63, 41, 10), (63, 80, 10),
          (63, 81, 20), (63, 159, 20), (16, 60, 2), (16, 61, 5), (16, 301, 20), (511, 1, 2),
          (511, 3, 5), (511, 6, 10), (511, 11, 20), (255, 4, 2), (255, 5, 5), (1, 512, 2),
          (1, 513, 5), (2, 850, 5), (2, 851, 10), (64, 14, 2), (64, 15, 5), (64, 71, 20)]


def say(*a):
    print(*a, file=sys.stderr, flush=True)


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available()
    return t


@pytest.fixture(scope="module")
def ctx(torch):
    c = cg.Context(device=0, arena_bytes=1 << 30)
    yield c
    c.close()


@pytest.mark.parametrize("nx,ny,rows", SHAPES)
@pytest.mark.parametrize("variant", (cg.CG_VARIANT_CLASSIC, cg.CG_VARIANT_PIPELINED))
def test_rows_bitwise(ctx, torch, nx, ny, rows, variant):
    info = ctx.cg_plan(nx, ny, variant)
    assert (info.path, info.seg_rows, info.seg_cols) == (2, rows, nx + 1)
    o = oracle.Order.segments(rows, info.lanes, info.seg_waves, info.seg_cols)
    rng = np.random.default_rng(nx * 1000 + ny)
    b = rng.uniform(-1, 1, (ny, nx))
    x0 = rng.uniform(-1, 1, (ny, nx))
    for m, start in ((1, None), (2, x0), (9, None), (23, x0)):
        say("on-chip rows", nx, ny, "variant", variant, "m", m, "x0", start is not None)
        kw = dict(tol=0.0, maxit=m, variant=variant)
        xo, ro = oracle.cg(b, nx, ny, mode=MODE_CANONICAL, order=o,
                           **(dict(kw, x0=start) if start is not None else kw))
        x = np.full_like(b, 7.0)
        rc, res = ctx.solve(b, x, nx, ny, **(dict(kw, x0=start) if start is not None else kw))
        assert (rc, res.iterations) == (ro.status, ro.iterations)
        np.testing.assert_array_equal(x, xo)
        assert res.rel_res_true == ro.rel_res_true
        # device vectors: with guards around x, x0 in x itself, and off the
        # 16-byte alignment
        buf = torch.full((nx * ny + 3,), 7.0, dtype=torch.float64, device="cuda")
        xd = buf[1:1 + nx * ny].view(ny, nx)
        bd = torch.from_numpy(b).cuda()
        if start is not None:
            xd.copy_(torch.from_numpy(start))
            kw = dict(kw, x0=xd)
        rc, res = ctx.solve(bd, xd, nx, ny, **kw)
        assert (rc, res.iterations) == (ro.status, ro.iterations)
        np.testing.assert_array_equal(xd.cpu().numpy(), xo)
        np.testing.assert_array_equal(bd.cpu().numpy(), b)
        assert buf[0] == 7.0 and bool((buf[1 + nx * ny:] == 7.0).all())


def test_zero_rhs_and_pinned_memory(ctx, torch):
    nx, ny = 33, 17
    z = torch.zeros((ny, nx), dtype=torch.float64, device="cuda")
    x = torch.full_like(z, 3.0)
    rc, res = ctx.solve(z, x, nx, ny, x0=x)
    assert rc == cg.CG_OK and res.iterations == 0 and not bool(x.any())
    # pinned host memory passed as host memory: the same answer as on the device
    b = np.random.default_rng(5).uniform(-1, 1, (ny, nx))
    bp = torch.from_numpy(b).pin_memory()
    xp = torch.zeros_like(bp).pin_memory()
    xd = torch.zeros_like(z)
    kw = dict(tol=1e-8, maxit=500)
    rc, rp = ctx.solve(bp, xp, nx, ny, **kw)
    rc2, rd = ctx.solve(torch.from_numpy(b).cuda(), xd, nx, ny, **kw)
    assert rc == rc2 == cg.CG_OK and rp.iterations == rd.iterations
    np.testing.assert_array_equal(xp.numpy(), xd.cpu().numpy())


@pytest.mark.parametrize("variant", (cg.CG_VARIANT_CLASSIC, cg.CG_VARIANT_PIPELINED))
def test_batch_of_forms(ctx, torch, variant):
    """One batch with solves of every form: each bitwise its own solve."""
    rng = np.random.default_rng(11)
    P, B, X, Y = [], [], [], []
    for nx, ny, _ in SHAPES:
        b = torch.from_numpy(rng.uniform(-1, 1, (ny, nx))).cuda()
        x, y = torch.zeros_like(b), torch.zeros_like(b)
        kw = dict(tol=0.0, maxit=17, variant=variant)
        ctx.solve(b, y, nx, ny, **kw)
        P.append(cg.make_problem(b, x, nx, ny, **kw))
        B.append(b), X.append(x), Y.append(y)
    ctx.cg_solve_batch(P)
    for x, y in zip(X, Y):
        assert torch.equal(x, y)
