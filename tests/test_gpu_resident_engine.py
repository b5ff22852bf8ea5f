"""Batches and served requests whose iterations run in the resident loop, where
the engine has to move a solve between the loop and its steps."""
import os
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


def context(arena=1 << 30, max_slots=0, **env):
    old = {k: os.environ.get(k) for k in env}
    os.environ.update({k: str(v) for k, v in env.items()})
    try:
        return cg.Context(device=0, arena_bytes=arena, max_slots=max_slots)
    finally:
        for k, v in old.items():
            if v is None:
                del os.environ[k]
            else:
                os.environ[k] = v


def rhs(torch, nx, ny, seed=1):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.rand(ny, nx, generator=g, device="cuda", dtype=torch.float64) * 2 - 1


@pytest.mark.parametrize("variant", [0, 1])
def test_no_room_for_the_tables_after_a_launch(torch, variant):
    """A solve that has run in the loop goes on by steps (odd chunks of them)
    when another solve's workspace leaves no room for the next launch's tables:
    the first solve's exchange area, then a workspace that ends within a few
    KiB of the arena, whatever the sizes of the engine's own tables."""
    nx, ny = 300, 190
    b = rhs(torch, nx, ny)
    first = dict(tol=0.0, maxit=3000, variant=variant)
    small, large = (64, 60), (64, 64)  # variable coefficients: they run by steps
    faces = {s: (torch.ones(s[1], s[0] + 1, device="cuda", dtype=torch.float64),
                 torch.ones(s[1] + 1, s[0], device="cuda", dtype=torch.float64))
             for s in (small, large)}
    with context(CG_RESIDENT=0) as c:
        x = torch.zeros_like(b)
        rc, ref = c.solve(b, x, nx, ny, **first)
        ref_x = x.cpu().numpy()
        need = c.cg_plan(nx, ny, variant).footprint + c.cg_plan(*large, 0, vc=True).footprint
    wgs = 3 * 12  # work-groups of the first solve's loop, two strips a wavefront
    need += 8 * (16 + 48 + 32 * wgs + 1024 * wgs + 128 * wgs)
    for spare in range(16 << 10, 64 << 10, 2 << 10):
        print("tables", variant, spare, flush=True)
        with context(arena=need + spare, max_slots=3, CG_STEP_CHUNK=7) as c:
            x = torch.zeros_like(b)
            probs = [cg.make_problem(b, x, nx, ny, **first)]
            keep = []
            for s, m in ((small, 40), (large, 400)):
                u, v = rhs(torch, *s), torch.zeros(s[1], s[0], device="cuda", dtype=torch.float64)
                keep += [u, v]
                probs.append(cg.make_problem(u, v, *s, tol=0.0, maxit=m, kx=faces[s][0],
                                             ky=faces[s][1]))
            rc, res = c.cg_solve_batch(probs)
            assert res[0].iterations == ref.iterations and res[0].status == ref.status
            assert res[0].rel_res_true == ref.rel_res_true
            np.testing.assert_array_equal(x.cpu().numpy(), ref_x)


@pytest.mark.parametrize("variant", [0, 1])
def test_a_small_solve_among_large_ones_gets_its_turn(torch, variant):
    """A request that one XCD holds is served long before requests that take
    the whole device, and that came first, are done; and one of those before
    the small requests that keep coming are."""
    n, m = 1024, 200
    big, small = rhs(torch, n, n), rhs(torch, m, m)
    xs = [torch.zeros_like(big) for _ in range(4)]
    x = torch.zeros_like(small)
    torch.cuda.synchronize()
    with context(arena=4 << 30) as c:
        def submit(b, x, side, **kw):
            return c.cg_submit(cg.make_problem(b, x, side, side, variant=variant, **kw))

        left = [submit(big, y, n, tol=0.0, maxit=6000) for y in xs]
        time.sleep(0.005)
        t = submit(small, x, m, tol=0.0, maxit=100)
        while c.cg_poll(t)[0] == cg.CG_PENDING:
            pass
        left = [t for t in left if c.cg_poll(t)[0] == cg.CG_PENDING]
        print("small solve done, large ones left:", len(left), flush=True)
        assert len(left) == 4
        turns = 0
        while left:
            t = submit(small, x, m, tol=0.0, maxit=100)
            while c.cg_poll(t)[0] == cg.CG_PENDING:
                left = [q for q in left if c.cg_poll(q)[0] == cg.CG_PENDING]
            turns += 1
            assert turns < 1000
