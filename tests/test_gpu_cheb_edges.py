"""GPU parity of the Chebyshev pass where its wavefronts (112 output columns of
128) and items (rows of a work-group) meet the edges of the grid: bitwise the
oracle's, at widths just below, at and above a wavefront's columns, odd and
even, and heights of one item and a remainder."""
import sys

import numpy as np
import pytest

import oracle
from oracle import MODE_CANONICAL
from paper_1803_03797_amd import cg

pytestmark = pytest.mark.gpu

WIDTHS = [3, 111, 112, 113, 120, 126, 127, 128, 129, 130, 223, 224, 231, 232, 233, 234, 240, 241,
          896, 898, 901]
HEIGHTS = [1, 2, 6, 7, 8, 14, 15, 16, 17, 22, 23, 24, 31, 33, 48, 50]


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


def check(ctx, nx, ny, s, variant, m):
    say("chebyshev edges", nx, ny, "s", s, "variant", variant, "m", m)
    info = ctx.cg_plan(nx, ny, variant=variant, precond=s)
    o = oracle.Order(info.cols_per_lane, info.lanes, info.waves, info.rows, info.threads2,
                     alt=info.walk_alt)
    orho = oracle.Order(2, info.lanes, 1, info.cheb_rows, info.threads2)
    b = np.random.default_rng(nx * 100 + ny).uniform(-1, 1, (ny, nx))
    x = np.zeros_like(b)
    rc, res = ctx.solve(b, x, nx, ny, tol=0.0, maxit=m, precond=s, variant=variant)
    xo, ro = oracle.pcg(b, nx, ny, s, tol=0.0, maxit=m, mode=MODE_CANONICAL, order=o,
                        order_rho=orho, variant=variant)
    assert (rc, res.iterations) == (ro.status, ro.iterations)
    np.testing.assert_array_equal(x, xo)
    assert res.rel_res_true == ro.rel_res_true


@pytest.mark.parametrize("nx", WIDTHS)
@pytest.mark.parametrize("s", (3, 5, 8))
def test_widths(ctx, nx, s):
    for ny, variant in ((33, cg.CG_VARIANT_CLASSIC), (16, cg.CG_VARIANT_PIPELINED)):
        check(ctx, nx, ny, s, variant, 3)


@pytest.mark.parametrize("ny", HEIGHTS)
@pytest.mark.parametrize("s", (4, 6, 7, 8))
def test_heights(ctx, ny, s):
    for nx, variant in ((234, cg.CG_VARIANT_CLASSIC), (113, cg.CG_VARIANT_PIPELINED)):
        check(ctx, nx, ny, s, variant, 3)


@pytest.mark.parametrize("nx,ny", [(113, 33), (128, 17), (130, 16), (241, 24), (898, 50)])
@pytest.mark.parametrize("s", (5, 7, 8))
def test_inner_solve_in_binary32(ctx, nx, ny, s):
    """The refinement's inner solve with the same pass: the tolerance on the
    true residual in binary64 is met, and the answer is the FP64 solve's within
    what two residuals of 1e-11 allow: |x - y| <= 2 tol |b| / lambda_min."""
    say("chebyshev binary32", nx, ny, "s", s)
    b = np.random.default_rng(nx + ny).uniform(-1, 1, (ny, nx))
    x, y = np.zeros_like(b), np.zeros_like(b)
    kw = dict(tol=1e-11, maxit=20000, precond=s)
    rc, res = ctx.solve(b, x, nx, ny, precision=cg.CG_PREC_FP32_REFINED, **kw)
    rc2, _ = ctx.solve(b, y, nx, ny, **kw)
    assert rc == rc2 == cg.CG_OK and res.rel_res_true <= 1e-11
    lmin = 4 * np.sin(np.pi / (2 * (nx + 1))) ** 2 + 4 * np.sin(np.pi / (2 * (ny + 1))) ** 2
    assert np.linalg.norm(x - y) <= 2.01e-11 * np.linalg.norm(b) / lmin
