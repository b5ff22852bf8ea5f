"""The autotuner and the resident loop: tuning a grid whose iterations run in
the loop does not put it back on passes, and neither does a cache line from
before shapes were measured against the loop."""
import json

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


def solve(torch, ctx, nx, ny, variant, prec):
    """(forms of the loop that ran, x, iterations)"""
    g = torch.Generator(device="cuda").manual_seed(1)
    b = torch.rand(ny, nx, generator=g, device="cuda", dtype=torch.float64) * 2 - 1
    x = torch.zeros_like(b)
    ctx.cg_kernel_stats(reset=True)
    _, r = ctx.solve(b, x, nx, ny, tol=1e-8, maxit=200, variant=variant, precision=prec)
    return sorted(ctx.cg_kernel_stats(reset=True)), x.cpu().numpy(), r.iterations


@pytest.mark.parametrize("nx,ny,variant,prec", [(300, 190, 0, 0), (512, 512, 1, 0),
                                                (1024, 1024, 1, 0), (1024, 1000, 0, 0),
                                                (600, 700, 0, cg.CG_PREC_FP32_REFINED)])
def test_a_tuned_grid_still_loops(torch, tmp_path, nx, ny, variant, prec):
    cache = str(tmp_path / "tune.json")
    with cg.Context(device=0, arena_bytes=1 << 30, tune_cache=cache) as c:
        forms, _, _ = solve(torch, c, nx, ny, variant, prec)
        assert len(forms) == 1 and forms[0].startswith("resident_")
        print("tune", nx, ny, variant, prec, flush=True)
        c.cg_set_profiling(True)  # the tuner's solves are timed as a caller runs them
        c.cg_tune(nx, ny, variant, prec)
        c.cg_set_profiling(False)
        tuned, x, its = solve(torch, c, nx, ny, variant, prec)
        assert len(tuned) == 1 and tuned[0].startswith("resident_")
    with cg.Context(device=0, arena_bytes=1 << 30, tune_cache=cache) as c:
        again, y, its2 = solve(torch, c, nx, ny, variant, prec)
        assert again == tuned and its == its2
        np.testing.assert_array_equal(x, y)


def test_cache_lines_from_before_the_loop(torch, tmp_path):
    """Such a line is ignored for a grid that loops and loaded for one that
    does not; a line that says "loop" is loaded for both."""
    cache = tmp_path / "tune.json"
    with cg.Context(device=0, arena_bytes=64 << 20, tune_cache=str(cache)) as c:
        c.cg_tune(300, 190)
        line = json.loads(open(cache).readline())
        assert line["loop"] == 1
    for loop in (0, 1):
        with open(cache, "w") as f:
            for n in (512, 2000):
                d = dict(line, nx=n, ny=n, variant=0, rows=16, grid=256, cpl=2)
                if not loop:
                    del d["loop"]
                f.write(json.dumps(d) + "\n")
        with cg.Context(device=0, arena_bytes=1 << 30, tune_cache=str(cache)) as c:
            assert c.cg_plan(2000, 2000).rows == 16
            assert (c.cg_plan(512, 512).rows == 16) == (loop == 1)
            forms, _, _ = solve(torch, c, 512, 512, 0, 0)
            assert forms == ([] if loop else ["resident_cg_2x4_near"])
