"""GPU parity of the sum over all tiles' partials at the counts where its
batches of loads end: bitwise the oracle's order, on the pass-by-pass path."""
import os
import sys

import numpy as np
import pytest

import oracle
from oracle import MODE_CANONICAL
from paper_1803_03797_amd import cg

pytestmark = pytest.mark.gpu

# 256 threads, 8 partials of one sum or 4 of two or three at a time
TILES = [383, 511, 512, 513, 767, 768, 769, 1023, 1024, 1025, 2047, 2048, 2049, 2305]


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available()
    old = {k: os.environ.get(k) for k in ("CG_RESIDENT", "CG_RR")}
    os.environ.update(CG_RESIDENT="0", CG_RR="0")
    try:
        c = cg.Context(device=0, arena_bytes=1 << 30)
    finally:
        for k, v in old.items():
            os.environ.pop(k, None) if v is None else os.environ.__setitem__(k, v)
    yield c
    c.close()


@pytest.mark.parametrize("tiles", TILES)
@pytest.mark.parametrize("variant,precond", [(cg.CG_VARIANT_CLASSIC, 0),
                                             (cg.CG_VARIANT_PIPELINED, 0),
                                             (cg.CG_VARIANT_PIPELINED, 2)])
def test_tile_counts(ctx, tiles, variant, precond):
    rows = 2
    nx, ny = 3, 4 * rows * tiles - 1
    ctx.cg_pin_tile(nx, ny, rows)
    info = ctx.cg_plan(nx, ny, variant=variant, precond=precond)
    print("cross-tile", tiles, "variant", variant, "precond", precond, "path", info.path,
          file=sys.stderr, flush=True)
    assert info.rows == rows and -(-ny // (info.waves * rows)) == tiles
    o = oracle.Order(info.cols_per_lane, info.lanes, info.waves, info.rows, info.threads2,
                     alt=info.walk_alt)
    b = np.random.default_rng(tiles).uniform(-1, 1, (ny, nx))
    x = np.zeros_like(b)
    kw = dict(tol=0.0, maxit=5, variant=variant)
    rc, res = ctx.solve(b, x, nx, ny, precond=precond, **kw)
    if precond:
        orho = oracle.Order(2, info.lanes, 1, info.cheb_rows, info.threads2)
        xo, ro = oracle.pcg(b, nx, ny, precond, mode=MODE_CANONICAL, order=o, order_rho=orho, **kw)
    else:
        xo, ro = oracle.cg(b, nx, ny, mode=MODE_CANONICAL, order=o, **kw)
    assert (rc, res.iterations) == (ro.status, ro.iterations)
    np.testing.assert_array_equal(x, xo)
    assert res.rel_res_recursive == ro.rel_res_recursive
    assert res.rel_res_true == ro.rel_res_true
