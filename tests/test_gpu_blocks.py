"""Blocks of right-hand sides in the operator calls: every block size gives each
right-hand side the bits of a call of its own (the default launch shape's fast
loop of 2 to 8 right-hand sides, and how larger calls are cut up)."""

import os
import subprocess
import sys

import numpy as np
import pytest

import synth
from tests.gpu_common import links, log, oracle_apply_A

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def stag():
    import paper_1111_0125_amd as s
    return s


@pytest.fixture(scope="module")
def ctx(stag):
    c = stag.Context(0)
    yield c
    c.close()


# 480 sites per parity: a half-filled last tile of links and last block
@pytest.mark.parametrize("n", [2, 3, 4, 5, 7, 8, 13, 16])
@pytest.mark.parametrize("prec,form", [("f64", "full"), ("f64", "r12"), ("f32", "full"), ("f32", "r12"),
                                       ("f16s", "full"), ("f16s", "r12"), ("f64", "improved"),
                                       ("f32", "improved"), ("f16s", "improved")])
def test_block_equals_singles(stag, ctx, n, prec, form):
    L = (6, 4, 4, 10)
    U = links(L, "haar", 81)
    lng = None
    if form == "improved":
        U, lng = synth.naik_links(U, fat_noise=0.05, seed=82)
    g = ctx.gauge(L, U, precisions=(prec,), r12=form == "r12", long=lng)
    v = synth.gaussian_rhs(L, n, 83)
    masses = [0.05 * (k + 1) for k in range(n)]
    fi, fo, ft = ctx.field(g, 0, prec, n).load(v), ctx.field(g, 0, prec, n), ctx.field(g, 1, prec, n)
    stag.stag_apply_A(ctx, g, masses, fi, fo)
    stag.stag_dslash(ctx, g, fi, ft)
    got, dgot = fo.store(), ft.store()
    f1, o1, t1 = ctx.field(g, 0, prec, 1), ctx.field(g, 0, prec, 1), ctx.field(g, 1, prec, 1)
    for k in range(n):
        f1.load(v[k:k + 1])
        stag.stag_apply_A(ctx, g, masses[k:k + 1], f1, o1)
        stag.stag_dslash(ctx, g, f1, t1)
        assert np.array_equal(o1.store()[0], got[k]), k
        assert np.array_equal(t1.store()[0], dgot[k]), k
    if form != "improved":
        ref = oracle_apply_A(U, v, L, masses)
        tol = {"f64": 1e-12, "f32": 1e-6, "f16s": 1e-3}[prec]
        assert np.abs(got - ref).max() <= tol * np.abs(ref).max()
    for o in (fi, fo, ft, f1, o1, t1, g):
        o.destroy()


@pytest.mark.parametrize("n", [3, 5, 6, 8, 11])
def test_block_solve_groups_equal_singles(stag, ctx, n):
    """Mixed solves of n right-hand sides, cut into groups (3; 4 + 4 with idle slots;
    8 + 3), with a kernel per stage: each has the bits of its own solve."""
    L = (8, 8, 8, 8)
    U = links(L, "exp", 84, 0.4)
    g = ctx.gauge(L, U, precisions=("f64", "f32"), r12=True)
    b = synth.gaussian_rhs(L, n, 85)
    masses = [0.1 + 0.01 * k for k in range(n)]
    fb, fx = ctx.field(g, 0, "f64", n).load(b), ctx.field(g, 0, "f64", n)
    p = stag.cg_params(tol=1e-9, inner="f32", small_lattice=False)
    rc, st = stag.stag_cg_solve(ctx, g, masses, fb, fx, p)
    assert rc == 0
    x = fx.store()
    f1, x1 = ctx.field(g, 0, "f64", 1), ctx.field(g, 0, "f64", 1)
    for k in (0, n // 2, n - 1):
        f1.load(b[k:k + 1])
        rc1, st1 = stag.stag_cg_solve(ctx, g, masses[k:k + 1], f1, x1, p)
        assert rc1 == 0 and st1[0]["iters"] == st[k]["iters"]
        assert np.array_equal(x1.store()[0], x[k]), k
    for o in (fb, fx, f1, x1, g):
        o.destroy()


@pytest.mark.parametrize("n", [12, 13, 16])
@pytest.mark.parametrize("form", ["full", "r12", "improved"])
def test_blocks_of_twelve_equal_singles(stag, ctx, n, form):
    """fp32 on 69984 sites per parity, where 12 to 15 right-hand sides take a block
    of 12 whole and 16 two of 8 (the improved operator on any lattice)."""
    L = (18, 18, 18, 24)
    U = links(L, "exp", 86, 0.4)
    lng = None
    if form == "improved":
        U, lng = synth.naik_links(U, fat_noise=0.05, seed=87)
    g = ctx.gauge(L, U, precisions=("f32",), r12=form == "r12", long=lng)
    v = synth.gaussian_rhs(L, n, 88)
    masses = [0.05 * (k + 1) for k in range(n)]
    fi, fo = ctx.field(g, 0, "f32", n).load(v), ctx.field(g, 0, "f32", n)
    stag.stag_apply_A(ctx, g, masses, fi, fo)
    got = fo.store()
    f1, o1 = ctx.field(g, 0, "f32", 1), ctx.field(g, 0, "f32", 1)
    for k in sorted({0, 7, 8, 11, n - 1}):
        f1.load(v[k:k + 1])
        stag.stag_apply_A(ctx, g, masses[k:k + 1], f1, o1)
        assert np.array_equal(o1.store()[0], got[k]), k
    for o in (fi, fo, f1, o1, g):
        o.destroy()


GROUPS = """
import sys
import torch
stream = torch.cuda.Stream() if sys.argv[1] == "torch" else None
import paper_1111_0125_amd as stag, synth
L = (16, 16, 16, 32)
with stag.Context(0) as ctx:
    g = ctx.gauge(L, synth.exp_ih_links(L, 89, 0.3), precisions=("f64", "f32"), r12=True)
    p = stag.cg_params(tol=1e-8, inner="f32", small_lattice=False)
    t = {}
    for n in (4, 8):
        fb = ctx.field(g, 0, "f64", n).load(synth.gaussian_rhs(L, n, 90))
        fx = ctx.field(g, 0, "f64", n)
        runs = [stag.stag_cg_solve(ctx, g, [0.2] * n, fb, fx, p, stream=stream) for _ in range(6)]
        assert all(rc == 0 for rc, st in runs)
        t[n] = min(st[0]["seconds"] for rc, st in runs)
print("RATIO", t[8] / t[4])
"""


@pytest.mark.parametrize("stream", ["torch", "own"])
def test_groups_overlap_whatever_else_uses_streams(stream):
    """8 right-hand sides on 16^3 x 32 run as two groups of 4 that overlap on the
    device (1.5 times the time of one group) in a program that creates streams of
    its own too; one after the other, as on streams that share a hardware queue,
    they take 2.1 times. (A program of its own: torch comes with its HIP runtime.)"""
    r = subprocess.run([sys.executable, "-c", GROUPS, stream], cwd=ROOT, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr
    ratio = float(r.stdout.split("RATIO")[1])
    log("groups, solves on stream:", stream, ratio)
    assert ratio < 1.85
