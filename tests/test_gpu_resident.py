"""The resident iteration loop (a mid-size solve's iterations in one launch) in
every compiled form against the same solve by passes, which the parity tests
hold to the oracle: same status, iteration count, residuals and x, bit for
bit."""
import os
import threading

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


@pytest.fixture(scope="module")
def passes(torch):
    with context(CG_RESIDENT=0) as c:
        yield c


def rhs(torch, nx, ny, seed=1):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.rand(ny, nx, generator=g, device="cuda", dtype=torch.float64) * 2 - 1


def solve(torch, ctx, b, x0=None, **kw):
    ny, nx = b.shape
    x = torch.zeros_like(b)
    rc, r = ctx.solve(b, x, nx, ny, x0=x0, **kw)
    return rc, r, x.cpu().numpy()


def same(a, b):
    assert a[0] == b[0] and a[1].status == b[1].status
    assert a[1].iterations == b[1].iterations
    assert a[1].outer_iterations == b[1].outer_iterations
    np.testing.assert_array_equal([a[1].rel_res_recursive, a[1].rel_res_true],
                                  [b[1].rel_res_recursive, b[1].rel_res_true])
    np.testing.assert_array_equal(a[2], b[2])


MODES = [(0, cg.CG_PREC_FP64), (1, cg.CG_PREC_FP64), (0, cg.CG_PREC_FP32_REFINED)]
# one tile column and many, ragged rows and columns, one strip of a tile in the
# grid, 256 tiles and one row of tiles more, more than 1024 tiles
SHAPES = [(129, 128), (300, 190), (257, 130), (17, 1100), (1100, 17), (130, 145), (512, 512),
          (512, 513), (1024, 1017), (1100, 1100), (600, 4), (2, 4000), (1, 5121)]


@pytest.mark.parametrize("strips", [0, 1, 2, 4])
@pytest.mark.parametrize("near", [0, 1])
def test_forms_equal_the_passes(torch, passes, strips, near):
    """Every number of strips, on one XCD and over all, launches of 7
    iterations and of many (a shape that a form does not fit runs by passes)."""
    with context(CG_RESIDENT_STRIPS=strips, CG_RESIDENT_NEAR=near) as c, \
            context(CG_RESIDENT_STRIPS=strips, CG_RESIDENT_NEAR=near, CG_RESIDENT_BUDGET=7) as s:
        for nx, ny in SHAPES:
            b = rhs(torch, nx, ny, nx + ny)
            for variant, prec in MODES:
                kws = [dict(tol=0.0, maxit=m) for m in (1, 2, 15)] if prec == 0 else []
                for kw in kws + [dict(tol=1e-8, maxit=60)]:
                    print("resident", strips, near, nx, ny, variant, prec, kw, flush=True)
                    ref = solve(torch, passes, b, variant=variant, precision=prec, **kw)
                    same(solve(torch, c, b, variant=variant, precision=prec, **kw), ref)
                    same(solve(torch, s, b, variant=variant, precision=prec, **kw), ref)


@pytest.mark.parametrize("variant,prec", MODES)
def test_natural_stop_and_warm_start(torch, passes, variant, prec):
    with context() as c:
        for nx, ny in ((300, 190), (2048, 2048) if prec else (700, 650)):
            b = rhs(torch, nx, ny, 3)
            x0 = rhs(torch, nx, ny, 4)
            for start in (None, x0):
                tol = 1e-4 if nx > 1000 else 1e-8
                print("natural stop", nx, ny, variant, prec, flush=True)
                kw = dict(tol=tol, maxit=20000, variant=variant, precision=prec, x0=start)
                ref = solve(torch, passes, b, **kw)
                assert ref[0] == cg.CG_OK
                same(solve(torch, c, b, **kw), ref)


@pytest.mark.parametrize("variant,prec", MODES)
def test_special_right_hand_sides(torch, passes, variant, prec):
    with context() as c:
        for what in ("zero", "nan", "inf", "huge", "tiny"):
            b = rhs(torch, 300, 190, 5)
            if what == "zero":
                b.zero_()
            elif what in ("nan", "inf"):
                b[60, 70] = float(what)
            else:
                b *= 1e200 if what == "huge" else 1e-200
            print("special", what, variant, prec, flush=True)
            kw = dict(tol=1e-8, maxit=50, variant=variant, precision=prec)
            same(solve(torch, c, b, **kw), solve(torch, passes, b, **kw))


def test_a_wait_given_up_runs_the_solve_by_passes(torch, passes):
    """One poll and no more: the solve is abandoned on the device and run by
    passes, with the same result."""
    with context(CG_RESIDENT_SPIN=1) as c:
        for variant, prec in MODES:
            b = rhs(torch, 640, 512, 6)
            print("given up", variant, prec, flush=True)
            kw = dict(tol=1e-8, maxit=300, variant=variant, precision=prec)
            for _ in range(2):
                same(solve(torch, c, b, **kw), solve(torch, passes, b, **kw))


def test_no_room_for_the_exchange_area(torch, passes):
    """An arena the solve just fits: accepted as ever, and run by passes."""
    b = rhs(torch, 640, 512, 7)
    ny, nx = b.shape
    with context() as c:
        need = c.cg_plan(nx, ny).footprint
    with context(arena=need) as c:
        kw = dict(tol=1e-8, maxit=100)
        same(solve(torch, c, b, **kw), solve(torch, passes, b, **kw))


def test_contexts_in_several_threads(torch, passes):
    """Launches whose work-groups wait for each other do not share the device."""
    cases = [(rhs(torch, 640, 512, 8 + k), k % 2) for k in range(4)]
    ref = [solve(torch, passes, b, tol=1e-6, maxit=5000, variant=v) for b, v in cases]
    torch.cuda.synchronize()
    got, errors = [None] * 4, []

    def work(k):
        try:
            with context() as c:
                for _ in range(3):
                    got[k] = solve(torch, c, cases[k][0], tol=1e-6, maxit=5000,
                                   variant=cases[k][1])
        except Exception as e:  # noqa: BLE001
            errors.append(e)

    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors
    for a, b in zip(got, ref):
        same(a, b)


# ------------------------------------------------ batches and serving --

# classic, pipelined and refined solves of one to many work-groups, a
# preconditioned, a 3D and a variable-coefficient one that step beside them,
# small ones that run whole, and one too large for one XCD
MIX = [(300, 190, 0, 0, 0), (300, 190, 1, 0, 0), (200, 180, 0, 1, 0), (129, 140, 0, 0, 0),
       (512, 512, 1, 0, 0), (513, 300, 0, 0, 0), (700, 600, 0, 1, 0), (100, 60, 0, 0, 0),
       (260, 260, 0, 0, 4), (17, 1100, 1, 0, 0), (1000, 37, 0, 0, 0), (900, 1000, 0, 1, 0),
       (640, 700, 0, 0, 0), (1024, 1024, 1, 0, 0), (150, 150, 0, 1, 0), (129, 128, 1, 0, 0)]


def mix(torch, tol=1e-6, maxit=4000):
    bs = [rhs(torch, nx, ny, 20 + k) for k, (nx, ny, _, _, _) in enumerate(MIX)]
    kw = [dict(tol=tol, maxit=maxit, variant=v, precision=p, precond=pc)
          for _, _, v, p, pc in MIX]
    return bs, kw


@pytest.fixture(scope="module")
def mix_alone(torch, passes):
    bs, kw = mix(torch)
    return [solve(torch, passes, b, **k) for b, k in zip(bs, kw)]


def as_batch(torch, ctx, bs, kws):
    xs = [torch.zeros_like(b) for b in bs]
    rc, res = ctx.cg_solve_batch([cg.make_problem(b, x, b.shape[1], b.shape[0], **k)
                                  for b, x, k in zip(bs, xs, kws)])
    return [(r.status, r, x.cpu().numpy()) for r, x in zip(res, xs)]


def as_served(torch, ctx, bs, kws):
    import time
    xs = [torch.zeros_like(b) for b in bs]
    tickets = [ctx.cg_submit(cg.make_problem(b, x, b.shape[1], b.shape[0], **k))
               for b, x, k in zip(bs, xs, kws)]
    out = [None] * len(bs)
    while any(o is None for o in out):
        for m, t in enumerate(tickets):
            if out[m] is None:
                rc, r = ctx.cg_poll(t)
                if rc != cg.CG_PENDING:
                    out[m] = (rc, cg.cg_result.from_buffer_copy(r))
        time.sleep(0.0005)
    return [(rc, r, x.cpu().numpy()) for (rc, r), x in zip(out, xs)]


@pytest.mark.parametrize("how", [as_batch, as_served])
@pytest.mark.parametrize("env", [{}, {"CG_RESIDENT_SPIN": 1}, {"CG_STEP_CHUNK": 7,
                                                               "CG_SERVE_CHUNK": 5}])
def test_engine_equals_the_passes(torch, mix_alone, how, env):
    """Many solves in the loop at once, then with every wait given up (all
    restart by steps), then with odd chunks of steps beside it."""
    bs, kws = mix(torch)
    with context(arena=4 << 30, **env) as c:
        print("engine", how.__name__, env, flush=True)
        for got, ref in zip(how(torch, c, bs, kws), mix_alone):
            same(got, ref)


def test_engine_with_more_solves_than_the_device_holds(torch, passes):
    bs = [rhs(torch, 480 + k, 500, 50 + k % 3) for k in range(20)]
    kws = [dict(tol=1e-3, maxit=2000, variant=k % 2) for k in range(20)]
    ref = [solve(torch, passes, b, **k) for b, k in zip(bs, kws)]
    for arena in (4 << 30, 200 << 20):
        with context(arena=arena) as c:
            print("many", arena, flush=True)
            for got, r in zip(as_batch(torch, c, bs, kws), ref):
                same(got, r)
