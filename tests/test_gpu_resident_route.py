"""Which solves run their iterations in the resident loop, and in which form.
The loop and the passes give the same bits, so only the context's statistics
tell them apart."""
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


def context(arena=1 << 30, **env):
    old = {k: os.environ.get(k) for k in env}
    os.environ.update({k: str(v) for k, v in env.items()})
    try:
        return cg.Context(device=0, arena_bytes=arena)
    finally:
        for k, v in old.items():
            if v is None:
                del os.environ[k]
            else:
                os.environ[k] = v


def rhs(torch, nx, ny, seed=1):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.rand(ny, nx, generator=g, device="cuda", dtype=torch.float64) * 2 - 1


def loops(ctx):
    """{form: launches} since the last call."""
    st = ctx.cg_kernel_stats(reset=True)
    assert all(s["seconds"] == 0 and s["bytes"] == 0 for s in st.values())
    return {k[len("resident_"):]: s["launches"] for k, s in st.items()}


def forms(torch, ctx, nx, ny, tol=0.0, maxit=20):
    """The forms of the classic, the pipelined and the refined solve."""
    b = rhs(torch, nx, ny)
    out = []
    for variant, prec in ((0, cg.CG_PREC_FP64), (1, cg.CG_PREC_FP64),
                          (0, cg.CG_PREC_FP32_REFINED)):
        loops(ctx)
        ctx.solve(b, torch.zeros_like(b), nx, ny, tol=1e-8 if prec else tol, maxit=maxit,
                  variant=variant, precision=prec)
        got = loops(ctx)
        assert len(got) <= 1, got
        out.append(next(iter(got), None))
    return out


# one XCD holds a solve or it takes them all; the grids after which solves run by
# passes; grids that never loop (on chip)
ROUTES = [((129, 128), ["cg_2x1_near", "pcg_2x1_near", "cg_f32_2x1_near"]),
          ((300, 190), ["cg_2x1_near", "pcg_2x1_near", "cg_f32_2x1_near"]),
          ((384, 384), ["cg_2x2_near", "pcg_2x1_far", "cg_f32_2x1_near"]),
          ((512, 512), ["cg_2x4_near", "pcg_2x2_far", "cg_f32_2x2_near"]),
          ((640, 512), ["cg_2x2_far", "pcg_2x2_far", "cg_f32_2x2_near"]),
          ((1024, 1024), ["cg_2x4_far", "pcg_2x4_far", "cg_f32_2x4_far"]),
          ((1025, 1024), ["cg_2x4_far", None, "cg_f32_2x4_far"]),
          ((1024, 1025), ["cg_2x4_far", None, "cg_f32_2x4_far"]),
          ((1536, 1025), ["cg_2x4_far", None, "cg_f32_2x4_far"]),
          ((1536, 1040), [None, None, "cg_f32_2x4_far"]),
          ((1234, 1234), ["cg_2x4_far", None, "cg_f32_2x4_far"]),
          ((1760, 1760), [None, None, "cg_f32_2x4_far"]),
          ((1764, 1764), [None, None, "cg_f32_3x6_far"]),
          ((2047, 2048), [None, None, "cg_f32_4x4_far"]),
          ((2048, 2047), [None, None, "cg_f32_3x6_far"]),
          ((2049, 2049), [None, None, "cg_f32_4x5_far"]),
          ((2240, 2240), [None, None, "cg_f32_4x5_far"]),
          ((2241, 2241), [None, None, None]),
          ((100, 100), [None, None, "cg_f32_2x1_near"])]


def test_routes(torch):
    with context() as c:
        for (nx, ny), want in ROUTES:
            print("route", nx, ny, flush=True)
            assert forms(torch, c, nx, ny) == want, (nx, ny)


@pytest.mark.parametrize("near", [0, 1])
@pytest.mark.parametrize("strips", [1, 2, 4])
def test_every_form_runs(torch, strips, near):
    with context(CG_RESIDENT_STRIPS=strips, CG_RESIDENT_NEAR=near) as c:
        print("form", strips, near, flush=True)
        end = "_2x%d_%s" % (strips, "near" if near else "far")
        # four strips of the pipelined solve: never on one XCD
        pcg = "pcg_2x4_far" if strips == 4 else "pcg" + end
        assert forms(torch, c, 129, 128) == ["cg" + end, pcg, "cg_f32" + end]


def test_launches(torch):
    """A launch runs its budget of iterations, and one more solve takes the
    same again."""
    nx, ny = 300, 190
    b = rhs(torch, nx, ny)
    with context(CG_RESIDENT_BUDGET=10) as c:
        for _ in range(2):
            c.solve(b, torch.zeros_like(b), nx, ny, tol=0.0, maxit=95)
            assert loops(c) == {"cg_2x1_near": 10}
    with context(CG_RESIDENT=0) as c:
        c.solve(b, torch.zeros_like(b), nx, ny, tol=0.0, maxit=95)
        assert loops(c) == {}


def test_abandoned_solves_are_counted(torch):
    for nx, ny in ((300, 190), (640, 512)):
        b = rhs(torch, nx, ny)
        with context(CG_RESIDENT_SPIN=1) as c:
            x = torch.zeros_like(b)
            c.solve(b, x, nx, ny, tol=0.0, maxit=200)
            assert loops(c)["abandoned"] == 1
        with context() as c:
            y = torch.zeros_like(b)
            c.solve(b, y, nx, ny, tol=0.0, maxit=200)
            assert "abandoned" not in loops(c)
            np.testing.assert_array_equal(x.cpu().numpy(), y.cpu().numpy())


def test_batches_loop(torch):
    """The solves of a batch loop, with none abandoned; with waits of one poll
    they are, and restart by steps."""
    shapes = [(300, 190, 0, 0), (384, 384, 1, 0), (512, 512, 0, 0), (700, 650, 0, 1),
              (1024, 1024, 1, 0), (129, 128, 1, 0)]
    bs = [rhs(torch, nx, ny) for nx, ny, _, _ in shapes]

    def batch(c):
        xs = [torch.zeros_like(b) for b in bs]
        c.cg_solve_batch([cg.make_problem(b, x, nx, ny, tol=1e-6, maxit=300, variant=v,
                                          precision=p)
                          for b, x, (nx, ny, v, p) in zip(bs, xs, shapes)])
        return [x.cpu().numpy() for x in xs]

    with context(arena=4 << 30) as c:
        want = batch(c)
        got = loops(c)
        print("batch", got, flush=True)
        assert "abandoned" not in got
        assert {k.rsplit("_", 2)[0] for k in got} == {"cg", "pcg", "cg_f32"}
        assert sum(got.values()) >= len(shapes)
        assert any(k.endswith("far") for k in got) and any(k.endswith("near") for k in got)
    with context(arena=4 << 30, CG_RESIDENT_SPIN=1) as c:
        for a, b in zip(batch(c), want):
            np.testing.assert_array_equal(a, b)
        assert 1 <= loops(c)["abandoned"] <= len(shapes)


@pytest.mark.parametrize("batch", [0, 1])
def test_the_loop_pauses_after_an_abandoned_solve(torch, batch):
    """What held the device is likely to stay: the next solves run by passes,
    without waiting for it each, until a pause of a second is over."""
    nx, ny = 640, 512
    b = rhs(torch, nx, ny)

    def run(c):
        x = torch.zeros_like(b)
        p = cg.make_problem(b, x, nx, ny, tol=0.0, maxit=50)
        if batch:
            c.cg_solve_batch([p])
        else:
            c.cg_solve(p)
        return x.cpu().numpy()

    with context(CG_RESIDENT=0) as c:
        want = run(c)
    with context(CG_RESIDENT_SPIN=1) as c:
        for n in (1, 1, 1):
            np.testing.assert_array_equal(run(c), want)
            assert c.cg_kernel_stats()["resident_abandoned"]["launches"] == n
        time.sleep(1.1)
        for n in (2, 2):
            np.testing.assert_array_equal(run(c), want)
            assert c.cg_kernel_stats()["resident_abandoned"]["launches"] == n


def test_no_gap_in_the_refined_range(torch):
    """Every refined square up to 2240 loops."""
    with context() as c:
        for n in list(range(150, 1700, 77)) + list(range(1700, 2241, 13)) + [2240]:
            b = torch.ones(n, n, device="cuda", dtype=torch.float64)
            loops(c)
            c.solve(b, torch.zeros_like(b), n, n, tol=1e-8, maxit=4,
                    precision=cg.CG_PREC_FP32_REFINED)
            got = loops(c)
            assert len(got) == 1 and "abandoned" not in got, (n, got)


# tall strips: their first and last grid, ragged rows and columns, one tile
# column and many, a last work-group of few strips
TALL = [(1764, 1764, "3x6"), (2041, 1805, "3x6"), (250, 13001, "3x6"), (2048, 2047, "3x6"),
        (4000, 1001, "3x6"), (2048, 2048, "4x4"), (1023, 4096, "4x4"), (2049, 2049, "4x5"),
        (2240, 2240, "4x5"), (3001, 1403, "4x5"), (255, 16399, "4x5")]


@pytest.mark.parametrize("nx,ny,form", TALL)
def test_tall_strips_equal_the_passes(torch, nx, ny, form):
    b, x0 = rhs(torch, nx, ny, nx), rhs(torch, nx, ny, ny)
    kw = dict(precision=cg.CG_PREC_FP32_REFINED)
    with context() as c, context(CG_RESIDENT_BUDGET=7) as s, context(CG_RESIDENT=0) as p:
        for start, tol, maxit in ((None, 1e-3, 90), (x0, 1e-8, 41)):
            print("tall", nx, ny, form, maxit, flush=True)
            out = []
            for ctx in (p, c, s):
                loops(ctx)
                x = torch.zeros_like(b)
                rc, r = ctx.solve(b, x, nx, ny, x0=start, tol=tol, maxit=maxit, **kw)
                assert list(loops(ctx)) == ([] if ctx is p else ["cg_f32_%s_far" % form])
                out.append((rc, r.iterations, r.outer_iterations, r.rel_res_true, x.cpu().numpy()))
            for o in out[1:]:
                assert o[:4] == out[0][:4]
                np.testing.assert_array_equal(o[4], out[0][4])
