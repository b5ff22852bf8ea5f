"""Batches and served requests whose iterations run in the resident loop, where
the engine has to move a solve between the loop and its steps."""
import os

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
