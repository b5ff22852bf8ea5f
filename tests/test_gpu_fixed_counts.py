"""GPU parity of the fixed-point solver at the unknown counts where the unknowns
per thread (1, 2, 3, 4, 6, 8, 10 of 1024 threads) change: every bit the
oracle's, alone and in one batch of all of them."""
import sys

import numpy as np
import pytest

from oracle import cg_fixed
from paper_1803_03797_amd import cg

pytestmark = pytest.mark.gpu

SHAPES = [(1, 63), (1, 64), (1, 65), (1, 1024), (1, 1025), (1, 2048), (1, 2049), (1, 3072),
          (1, 3073), (1, 4096), (1, 4097), (1, 5121), (1, 6144), (1, 6145), (128, 64), (3, 2731),
          (96, 96)]
VARIANTS = (cg.CG_VARIANT_CLASSIC, cg.CG_VARIANT_PIPELINED)


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available()
    c = cg.Context(device=0, arena_bytes=1 << 30)
    yield c
    c.close()


def rhs(nx, ny):
    # from small values to ones whose products saturate
    rng = np.random.default_rng(nx * ny)
    return rng.uniform(-1, 1, (ny, nx)) * 10.0 ** rng.integers(-6, 6, (ny, nx))


@pytest.mark.parametrize("variant", VARIANTS)
def test_counts(ctx, variant):
    P, X, want = [], [], []
    for nx, ny in SHAPES:
        print("fixed counts", nx, ny, "variant", variant, file=sys.stderr, flush=True)
        for b in (rhs(nx, ny), np.random.default_rng(nx + ny).uniform(-1, 1, (ny, nx))):
            kw = dict(variant=variant, tol=0.0, maxit=12)
            xo, _, ro = cg_fixed(b, nx, ny, **kw)
            x = np.zeros_like(b)
            rc, res = ctx.solve(b, x, nx, ny, precision=cg.CG_PREC_FIXED, **kw)
            assert (rc, res.iterations) == (ro.status, ro.iterations)
            np.testing.assert_array_equal(x, xo)
            y = np.zeros_like(b)
            P.append(cg.make_problem(b, y, nx, ny, precision=cg.CG_PREC_FIXED, **kw))
            X.append((b, y))
            want.append(xo)
    ctx.cg_solve_batch(P)
    for (_, y), xo in zip(X, want):
        np.testing.assert_array_equal(y, xo)
