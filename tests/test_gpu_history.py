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


def test_tape_memory_is_reused_and_given_back():
    """Tapes of growing and shrinking sizes and two at a time, in memory kept of earlier ones, give the results of a
    fresh context bit for bit; trim gives the memory back."""
    import torch
    import paper_2206_02362_amd as fw
    ctx = fw.Context(0)

    def problem(nz, nshots, seed):
        w = synth.tiny(nz=nz, nx=70, nb=9, nt=181, nshots=nshots, nh=5, seed=seed)
        grid, tv, tg = gpu_problem(w)
        pt = _dev(0.2 * synth.random_ptilde(5, nz, 70, seed))
        return grid, tg, tv.clone().requires_grad_(True), pt.requires_grad_(True)

    def grads(q, c, pred=None):
        grid, tg, v, p = q
        pred = fw.predicted_data(v, p, c, grid, tg) if pred is None else pred
        return [pred.detach()] + list(torch.autograd.grad(pred.square().sum(), (v, p)))

    qs = [problem(40, 2, 1), problem(60, 6, 2), problem(57, 3, 3)]
    want = []
    for q in qs:
        c = fw.Context(0)
        want.append(grads(q, c))
        c.close()
    for i in (0, 1, 2, 0, 1):
        assert all(torch.equal(a, b) for a, b in zip(grads(qs[i], ctx), want[i])), i
    both = [fw.predicted_data(q[2], q[3], ctx, q[0], q[1]) for q in (qs[2], qs[1])]
    for i, pred in zip((2, 1), both):
        assert all(torch.equal(a, b) for a, b in zip(grads(qs[i], ctx, pred), want[i])), i
    assert ctx.info()["tape_bytes"] == 0
    big = 6 * 180 * 78 * 128 * 4                 # at least one T2 history of the largest problem
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    ctx.trim()
    assert torch.cuda.mem_get_info()[0] >= before + big
    ctx.close()


@pytest.mark.parametrize("nz,nx,nt,nshots,nh", [(57, 33, 158, 24, 5), (40, 50, 301, 2, 19)])
def test_vp_step_bits_do_not_depend_on_the_store(nz, nx, nt, nshots, nh):
    """The solver's images are summed in one order whether the background is kept whole or checkpointed."""
    import paper_2206_02362_amd as fw
    w = synth.tiny(nz=nz, nx=nx, nb=8, nt=nt, nshots=nshots, nh=nh, seed=6)
    grid, tv, tg = gpu_problem(w)
    got = []
    for budget in (0, 1 << 30):
        ctx = fw.Context(0, hbm_budget_bytes=budget)
        dobs = 0.7 * ctx.model(grid, tv, tg)
        p, phi = ctx.vp_solve(grid, tv, tg, dobs, nh, 1e-3, synth.dso_weights(nh), 3)
        got.append((p.cpu().numpy(), np.asarray(phi)))
        ctx.close()
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])


@pytest.mark.parametrize("nz,nx,nb,nt,nshots,nh", [(24, 32, 8, 3, 2, 5), (57, 33, 5, 158, 24, 5), (40, 50, 8, 301, 1, 19),
                                                   (60, 70, 9, 181, 3, 37)])
def test_bits_do_not_depend_on_the_store(nz, nx, nb, nt, nshots, nh):
    """Images and gradient sums are formed per checkpointed segment, from the last to the first, whether the wavefields'
    T2 terms are kept whole or recomputed: no FP32 sum is longer than a checkpointed segment's."""
    import torch
    import paper_2206_02362_amd as fw
    print(f"case: bits of history and checkpoints {nz}x{nx} nt{nt} {nshots} shots nh{nh}", file=sys.stderr, flush=True)
    w = synth.tiny(nz=nz, nx=nx, nb=nb, nt=nt, nshots=nshots, nh=nh, seed=14)
    grid, tv, tg = gpu_problem(w)
    pt = _dev(0.2 * synth.random_ptilde(nh, nz, nx, 5))
    data = _dev(np.random.default_rng(6).standard_normal((nshots, w.nrec, nt)))
    got = []
    for budget in (0, 1 << 30):
        ctx = fw.Context(0, hbm_budget_bytes=budget)
        v, p = tv.clone().requires_grad_(True), pt.clone().requires_grad_(True)
        pred = fw.predicted_data(v, p, ctx, grid, tg)
        got.append([pred.detach(), *torch.autograd.grad(0.5 * (pred - data).square().sum(), (v, p)),
                    *ctx.gradient(grid, tv, tg, pt, data, 1e-3, synth.dso_weights(nh)),
                    ctx.born_ext_fwd(grid, tv, tg, pt), ctx.born_ext_adj(grid, tv, tg, data, nh)])
        ctx.close()
    for a, b in zip(*got):
        assert torch.equal(a, b)


def test_histories_in_several_batches():
    """Where not all shots' histories fit the third of the device, those of large batches do: two batches of 30 shots (1920
    two-step workgroups) against one checkpointed batch, on a device with 14 GiB left."""
    import torch
    import paper_2206_02362_amd as fw
    print("case: histories in two batches, 60x1000 nt40 60 shots", file=sys.stderr, flush=True)
    nh, n = 5, 60
    w = synth.tiny(nz=60, nx=1000, nb=8, nt=40, nshots=n, nh=nh, seed=9)
    grid, tv, tg = gpu_problem(w)
    pt = _dev(0.2 * synth.random_ptilde(nh, 60, 1000, 3))
    data = _dev(np.random.default_rng(4).standard_normal((n, w.nrec, 40)))
    gib, got = 1 << 30, []
    for budget in (0, 6 * gib):
        torch.cuda.empty_cache()
        ctx = fw.Context(0, hbm_budget_bytes=budget)
        hold = torch.empty(max(0, torch.cuda.mem_get_info()[0] - 14 * gib), dtype=torch.uint8, device="cuda:0")
        got.append([*ctx.gradient(grid, tv, tg, pt, data, 1e-3, synth.dso_weights(nh)),
                    ctx.born_ext_adj(grid, tv, tg, data, nh)])
        got[-1].append(ctx.held_bytes() / gib)
        ctx.close()
        del hold
    torch.cuda.empty_cache()
    assert 4.2 < got[0][-1] < 4.8 and got[1][-1] < 3.0      # whole for all 60 shots: 4.85; checkpointed: 2.2
    for a, b in zip(got[0][:-1], got[1][:-1]):
        assert _close(_np(a), _np(b), 2e-6)
