"""Whole T2 histories against checkpointing.

A context without a budget keeps the T2 terms of every step where they fit; one
with a budget checkpoints and recomputes.  Both run the same propagations, so
their results differ by the order of the FP32 image sums only (a few units of
2^-24 of sums of a few thousand terms: 2e-6), and both match the oracle at the
suite's 1e-4.  Records of one step, odd ones, and shot counts that split the
record into several history segments.
"""
import sys

import numpy as np
import pytest

import oracle
import synth
from _helpers import gpu_problem, oracle_problem_f32, rel_l2

pytestmark = pytest.mark.gpu


def _dev(a):
    import torch
    return torch.tensor(np.asarray(a), dtype=torch.float32, device="cuda:0")


def _np(t):
    return t.detach().double().cpu().numpy()


def _close(a, b, tol):
    a, b = np.asarray(a), np.asarray(b)
    return np.linalg.norm((a - b).ravel()) <= tol * np.linalg.norm(b.ravel())


@pytest.mark.parametrize("nz,nx,nb,nt,nshots,nh", [(24, 32, 8, 2, 1, 1), (24, 32, 8, 3, 2, 5), (57, 33, 5, 158, 24, 5),
                                                   (60, 70, 9, 181, 3, 19)])
def test_history_and_checkpoints_agree(nz, nx, nb, nt, nshots, nh):
    import torch
    import paper_2206_02362_amd as fw
    print(f"case: history vs checkpoints {nz}x{nx} nb{nb} nt{nt} {nshots} shots nh{nh}", file=sys.stderr, flush=True)
    w = synth.tiny(nz=nz, nx=nx, nb=nb, nt=nt, nshots=nshots, nh=nh, seed=12)
    g, geo, vel = oracle_problem_f32(w)
    grid, tv, tg = gpu_problem(w)
    pt = (0.2 * synth.random_ptilde(nh, nz, nx, 3)).astype(np.float32)
    data = np.random.default_rng(4).standard_normal((nshots, w.nrec, nt)).astype(np.float32)
    dobs = (0.7 * oracle.model(g, vel, geo)).astype(np.float32)
    dso = synth.dso_weights(nh)
    got = []
    for budget in (0, 1 << 30):
        ctx = fw.Context(0, hbm_budget_bytes=budget)
        v, p = tv.clone().requires_grad_(True), _dev(pt).requires_grad_(True)
        pred = fw.predicted_data(v, p, ctx, grid, tg)
        gv, gp = torch.autograd.grad(0.5 * (pred - _dev(dobs)).square().sum(), (v, p))
        obj, gv2, gp2 = ctx.gradient(grid, tv, tg, _dev(pt), _dev(dobs), 1e-3, dso)
        pv, phi = ctx.vp_solve(grid, tv, tg, _dev(dobs), nh, 1e-3, dso, 2)
        got.append([_np(t) for t in (ctx.born_ext_fwd(grid, tv, tg, _dev(pt)),
                                     ctx.born_ext_adj(grid, tv, tg, _dev(data), nh), pred, gv, gp, obj, gv2, gp2, pv)]
                   + [np.asarray(phi)])
        ctx.close()
    for a, b in zip(*got):
        assert np.isfinite(a).all() and _close(a, b, 2e-6)
    p64, d64 = pt.astype(np.float64), data.astype(np.float64)
    ref = [oracle.born_ext_fwd(g, vel, geo, p64), oracle.born_ext_adj(g, vel, geo, d64, nh)]
    _, rv, rp = oracle.gradient(g, vel, geo, p64, dobs.astype(np.float64), 1e-3, dso)
    for a, b in zip([got[0][0], got[0][1], got[0][6], got[0][7]], ref + [rv, rp]):
        assert _close(a, b, 1e-4)
