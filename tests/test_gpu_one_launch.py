"""Calls that take one launch up to a bound on their sizes, on both sides of it.

* S and S* with the nodes in the launch (at most 384 nodes, 2048 rows, x cells of
  256 columns) and with tables in memory, against the oracle: sums of at most a
  few hundred FP32 terms, 1e-5 relative;
* the L-BFGS direction from inner products (at most 15 pairs) and by the
  recursion on vectors, against the oracle at that suite's 1e-5;
* input validation over more arrays than one launch takes, and non-finite
  values anywhere in an array.
"""
import sys

import numpy as np
import pytest

import oracle
import synth
from _helpers import gpu_problem, rel_l2

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2206_02362_amd as fw
    c = fw.Context(0)
    yield c
    c.close()


def dev(a):
    import torch
    return torch.tensor(np.asarray(a), dtype=torch.float32, device="cuda:0")


def t2n(t):
    return t.detach().double().cpu().numpy()


def _nodes(n, h, count, seed):
    """`count` nodes on [0, (n - 1) h], unevenly spaced."""
    rng = np.random.default_rng(seed)
    inner = np.sort(rng.choice(np.arange(1, 4 * (n - 1)), count - 2, replace=False)) if count > 2 else np.empty(0)
    return np.concatenate([[0.0], inner / 4.0, [n - 1.0]]) * h


@pytest.mark.parametrize("nz,nx,nzn,nxn", [(1, 1, 2, 2), (2, 257, 2, 2), (40, 259, 5, 2), (50, 700, 64, 4),
                                           (200, 330, 184, 200), (200, 330, 185, 200), (2048, 9, 30, 3),
                                           (2049, 9, 30, 3)])
def test_spline_bounds(ctx, nz, nx, nzn, nxn):
    print(f"case: spline {nz}x{nx} nodes {nzn}x{nxn}", file=sys.stderr, flush=True)
    dz, dx = 12.5, 10.0
    zn = _nodes(nz, dz, nzn, 1) if nz > 1 else np.array([0.0, 1.0])
    xn = _nodes(nx, dx, nxn, 2) if nx > 1 else np.array([0.0, 1.0])
    rng = np.random.default_rng(3)
    mc, f = rng.standard_normal((xn.size, zn.size)), rng.standard_normal((nx, nz))
    mc, f = mc.astype(np.float32), f.astype(np.float32)
    s = t2n(ctx.spline_apply(nz, nx, dz, dx, zn, xn, dev(mc)))
    a = t2n(ctx.spline_adjoint(nz, nx, dz, dx, zn, xn, dev(f)))
    assert rel_l2(s, oracle.spline_apply(zn, xn, nz, nx, dz, dx, mc)) < 1e-5
    assert rel_l2(a, oracle.spline_adjoint(zn, xn, nz, nx, dz, dx, f)) < 1e-5


@pytest.mark.parametrize("n,k", [(1, 1), (63, 2), (64, 3), (513, 4), (100_003, 14), (3001, 15), (3001, 16)])
def test_lbfgs_direction_bounds(ctx, n, k):
    print(f"case: lbfgs direction n {n}, {k} pairs", file=sys.stderr, flush=True)
    rng = np.random.default_rng(n + k)
    s = rng.standard_normal((k, n)).astype(np.float32)
    y = (s * rng.uniform(0.5, 2.0, n)).astype(np.float32)
    g = rng.standard_normal(n).astype(np.float32)
    ref = -oracle.two_loop(g.astype(np.float64), list(s.astype(np.float64)), list(y.astype(np.float64)))
    assert rel_l2(t2n(ctx.lbfgs_direction(dev(s), dev(y), dev(g))), ref) < 1e-5


def test_validation_of_many_arrays(ctx):
    import paper_2206_02362_amd as fw
    w = synth.tiny(nz=20, nx=30, nb=6, nt=40, nshots=1, seed=2)
    grid, tv, tg = gpu_problem(w)
    one = t2n(ctx.model(grid, tv, tg))
    out = ctx.model_batch([(grid, tv, tg)] * 70)            # 140 arrays
    assert all(np.array_equal(t2n(o), one) for o in out)
    for at in (0, 255, 599):                                # a velocity of the last job
        bad = tv.clone()
        bad.view(-1)[at] = float("nan")
        with pytest.raises(fw.FwimeError):
            ctx.model_batch([(grid, tv, tg)] * 69 + [(grid, bad, tg)])
    fast = tv.clone()
    fast.view(-1)[-1] = 1e5                                 # violates the CFL limit
    with pytest.raises(fw.FwimeError):
        ctx.model_batch([(grid, fast, tg)] + [(grid, tv, tg)] * 69)
