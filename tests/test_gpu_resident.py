"""Solves whose iterations run in the resident kernel (small lattices) against
the kernel-per-stage solver: the stages, their rounding and the reduction
order are the same, so the iterates are the same bits."""

import threading

import numpy as np
import pytest

import synth
from tests.gpu_common import links, log, oracle_apply_A

pytestmark = pytest.mark.gpu

# sites per parity: 192 (part of a block), 648 (a last wavefront of 8 sites), 2048, 3360,
# 16384 / 32768 / 65536 (the most for four, two and one lanes per site), and two above
LATTICES = [(4, 4, 4, 6), (6, 6, 6, 6), (8, 8, 8, 8), (8, 6, 10, 14), (16, 16, 16, 8),
            (16, 16, 16, 16), (16, 16, 16, 18), (16, 16, 16, 32)]


@pytest.fixture(scope="module")
def stag():
    import paper_1111_0125_amd as s
    return s


@pytest.fixture(scope="module")
def ctx(stag):
    c = stag.Context(0)
    yield c
    c.close()


def both(stag, ctx, g, b, masses, x0=None, **kw):
    n = b.shape[0]
    fb = ctx.field(g, 0, "f64", n).load(b)
    fx = ctx.field(g, 0, "f64", n)
    got = []
    for small in (True, False):
        if x0 is not None:
            fx.load(x0)
        rc, st = stag.stag_cg_solve(ctx, g, masses, fb, fx,
                                    stag.cg_params(small_lattice=small, use_x0=x0 is not None, **kw))
        got.append((rc, [(s["iters"], s["reliable_updates"], s["restarts"], s["true_rel_res"]) for s in st],
                    fx.store()))
    fb.destroy()
    fx.destroy()
    return got


@pytest.mark.parametrize("L", LATTICES)
@pytest.mark.parametrize("inner", ["f64", "f32", "f16s"])
@pytest.mark.parametrize("r12", [False, True])
def test_resident_equals_kernel_per_stage(stag, ctx, L, inner, r12):
    vh = L[0] * L[1] * L[2] * L[3] // 2
    U = links(L, "exp", 51, 0.3)
    g = ctx.gauge(L, U, precisions=("f64", "f32", "f16s"), r12=r12)
    n = 1 if vh > 4096 else 3
    masses = [0.2, 0.3, 0.25][:n]
    b = synth.gaussian_rhs(L, n, 52)
    print("resident", L, inner, r12, n, flush=True)
    (rc1, st1, x1), (rc2, st2, x2) = both(stag, ctx, g, b, masses, tol=1e-9, inner=inner)
    log("resident", L, inner, r12, st1)
    assert rc1 == 0 and rc2 == 0
    assert st1 == st2
    assert np.array_equal(x1, x2)
    if vh <= 4096:
        r = b - oracle_apply_A(U, x1, L, masses)
        assert max(np.linalg.norm(r[k]) / np.linalg.norm(b[k]) for k in range(n)) <= 1e-9
    g.destroy()


@pytest.mark.parametrize("inner", ["f64", "f32"])
@pytest.mark.parametrize("n", [2, 9, 16])
def test_resident_blocks_start_guess_and_cap(stag, ctx, inner, n):
    """Several right-hand sides (each its own group of blocks), a zero one, a
    start from a guess, and the iteration cap."""
    L = (6, 6, 6, 6)
    U = links(L, "haar", 53)
    g = ctx.gauge(L, U, precisions=("f64", "f32"))
    masses = [0.1 + 0.02 * k for k in range(n)]
    b = synth.gaussian_rhs(L, n, 54)
    b[n // 2] = 0.0
    x0 = synth.gaussian_rhs(L, n, 55)
    for kw in (dict(), dict(x0=x0), dict(max_iter=7, x0=x0)):
        print("resident block", inner, n, sorted(kw), flush=True)
        (rc1, st1, x1), (rc2, st2, x2) = both(stag, ctx, g, b, masses, tol=1e-10, inner=inner, **kw)
        assert rc1 == rc2 and st1 == st2
        assert np.array_equal(x1, x2)
        if "max_iter" not in kw:
            assert rc1 == 0
    g.destroy()


@pytest.mark.parametrize("variant", ["restart", "reliable", "fold_only"])
def test_resident_mixed_variants(stag, ctx, variant):
    L = (8, 8, 4, 8)
    U = links(L, "exp", 56, 0.4)
    g = ctx.gauge(L, U, precisions=("f64", "f32"))
    b = synth.gaussian_rhs(L, 1, 57)
    (rc1, st1, x1), (rc2, st2, x2) = both(stag, ctx, g, b, [0.1], tol=1e-9, inner="f32",
                                          mixed_variant=variant, max_iter=400)
    assert rc1 == rc2 and st1 == st2
    assert np.array_equal(x1, x2)
    g.destroy()


@pytest.mark.parametrize("inner", ["f64", "f32", "f16s"])
@pytest.mark.parametrize("r12", [False, True])
def test_which_lattices_are_solved_in_the_resident_kernel(stag, ctx, inner, r12):
    """Up to 65536 sites per parity, plain CG up to 32768 (two lanes per site), and
    no more workgroups than compute units; small_lattice=False never."""
    for L, n in [((4, 4, 4, 6), 16), ((6, 6, 6, 6), 1), ((8, 6, 10, 14), 2), ((16, 16, 16, 16), 1),
                 ((16, 16, 16, 18), 1), ((16, 16, 16, 32), 1), ((16, 16, 16, 32), 2),
                 ((16, 16, 16, 34), 1)]:
        vh = L[0] * L[1] * L[2] * L[3] // 2
        fits = n * vh <= (32768 if inner == "f64" else 65536)
        g = ctx.gauge(L, links(L, "exp", 58, 0.2), precisions=("f64", "f32", "f16s"), r12=r12)
        fb = ctx.field(g, 0, "f64", n).load(synth.gaussian_rhs(L, n, 59))
        fx = ctx.field(g, 0, "f64", n)
        for small in (True, False):
            before = stag.stag_resident_counts(ctx)
            rc, st = stag.stag_cg_solve(ctx, g, [0.5] * n, fb, fx,
                                        stag.cg_params(tol=1e-6, inner=inner, small_lattice=small))
            after = stag.stag_resident_counts(ctx)
            assert rc == 0
            assert after == (before[0] + (1 if fits and small else 0), before[1]), (L, n, small)
        for o in (fb, fx, g):
            o.destroy()


@pytest.mark.parametrize("inner", ["f64", "f32", "f16s"])
@pytest.mark.parametrize("n,guess", [(1, False), (3, False), (1, True), (3, True)])
def test_waits_that_run_out_fall_back_to_stages(stag, inner, n, guess):
    """With no wait granted every workgroup leaves at once; the solve starts over
    with a kernel per stage and has its bits, also from a guess. Later solves of
    the context keep to stages until the wait is set again, and are right."""
    L = (8, 8, 8, 8)
    U = links(L, "exp", 60, 0.3)
    b = synth.gaussian_rhs(L, n, 61)
    x0 = synth.gaussian_rhs(L, n, 62) if guess else None
    masses = [0.2, 0.3, 0.25][:n]
    with stag.Context(0) as c:
        g = c.gauge(L, U, precisions=("f64", "f32", "f16s"))
        stag.stag_resident_wait(c, -1.0)
        (rc1, st1, x1), (rc2, st2, x2) = both(stag, c, g, b, masses, x0=x0, tol=1e-9, inner=inner)
        assert stag.stag_resident_counts(c) == (1, 1)
        assert rc1 == rc2 == 0 and st1 == st2 and np.array_equal(x1, x2)
        (rc1, st1, x1), _ = both(stag, c, g, b, masses, x0=x0, tol=1e-9, inner=inner)
        assert stag.stag_resident_counts(c) == (1, 1)
        assert rc1 == 0 and np.array_equal(x1, x2)
        stag.stag_resident_wait(c, 2.0)
        (rc1, st1, x1), _ = both(stag, c, g, b, masses, x0=x0, tol=1e-9, inner=inner)
        assert stag.stag_resident_counts(c) == (2, 1)
        assert rc1 == 0 and st1 == st2 and np.array_equal(x1, x2)


def test_small_solves_of_several_threads_share_the_device(stag):
    """Four threads, each with a context of its own: 2 to 6 workgroups a solve, so
    all of them fit beside each other. Every solve starts in a resident kernel,
    no wait runs out, and each has the bits of the solve alone."""
    jobs = [((4, 4, 4, 4), "f64", False), ((6, 6, 6, 6), "f32", True), ((4, 4, 4, 4), "f64", True),
            ((4, 4, 4, 8), "f32", False)]
    solves, got, errors = 6, {}, []

    def work(key, job, n):
        try:
            L, inner, r12 = job
            with stag.Context(0) as c:
                g = c.gauge(L, links(L, "haar", 63), precisions=("f64", "f32"), r12=r12)
                fb = c.field(g, 0, "f64", 1).load(synth.gaussian_rhs(L, 1, 64))
                fx = c.field(g, 0, "f64", 1)
                xs = []
                for _ in range(n):
                    rc, st = stag.stag_cg_solve(c, g, [0.05], fb, fx, stag.cg_params(tol=1e-10, inner=inner))
                    assert rc == 0
                    xs.append(fx.store())
                got[key] = (xs, stag.stag_resident_counts(c))
        except BaseException as e:
            errors.append(e)

    for k, job in enumerate(jobs):
        work(("alone", k), job, 1)
    threads = [threading.Thread(target=work, args=(("together", k), job, solves)) for k, job in enumerate(jobs)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for k in range(len(jobs)):
        xs, counts = got["together", k]
        assert counts == (solves, 0)
        for x in xs:
            assert np.array_equal(x, got["alone", k][0][0])


@pytest.mark.parametrize("inner", ["f64", "f32", "f16s"])
def test_links_of_all_ones_bytes_end_as_by_stages(stag, inner):
    """Memory filled with ones is a NaN whose bits mark an empty word in the
    resident kernel: the solve ends as with a kernel per stage (breakdown in fp64
    and fp32), and no wait runs out."""
    L = (8, 8, 4, 8)
    U = links(L, "haar", 65).copy()
    U.view(np.uint64)[...] = np.uint64(0xFFFFFFFFFFFFFFFF)
    b = synth.gaussian_rhs(L, 1, 66)
    with stag.Context(0) as c:
        g = c.gauge(L, U, precisions=("f64", "f32", "f16s"))
        fb, fx = c.field(g, 0, "f64", 1).load(b), c.field(g, 0, "f64", 1)
        res = [stag.stag_cg_solve(c, g, [0.2], fb, fx, stag.cg_params(tol=1e-8, inner=inner, escalate=False,
                                                                      max_iter=50, small_lattice=small))
               for small in (True, False)]
        (rc1, st1), (rc2, st2) = res
        log("all ones", inner, res)
        assert rc1 == rc2 and st1[0]["iters"] == st2[0]["iters"]
        if inner != "f16s":
            assert rc1 == stag.STAG_EBREAKDOWN
        assert stag.stag_resident_counts(c) == (1, 0)
