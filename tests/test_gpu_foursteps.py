"""Four time steps per launch against two (FWIME_STEPS) and against the oracle.

Both kernels apply the same operations per cell: FP32 modeling and the gradient
agree bit for bit; the extended-precision Born pair agrees to the rounding of
its FP64 update (1e-7 of the result).  Records that end in launches of one to
four steps, grids at and off the 40-row tiles and both tile widths, receivers
that share cells, a free surface near tile boundaries.
"""
import os
import sys

import numpy as np
import pytest

import oracle
import synth
from _helpers import gpu_problem, oracle_problem_f32, rel_l2

pytestmark = pytest.mark.gpu


def _ctx(steps):
    import paper_2206_02362_amd as fw
    os.environ["FWIME_STEPS"] = str(steps)
    try:
        return fw.Context(0)
    finally:
        del os.environ["FWIME_STEPS"]


def _dev(a):
    import torch
    return torch.tensor(np.asarray(a), dtype=torch.float32, device="cuda:0")


def _np(t):
    return t.detach().double().cpu().numpy()


# (nz, nx, nb, nt, shots, free surface); 230 columns and 3 shots take the wider tiles
CASES = [(24, 32, 8, nt, 1, False) for nt in (2, 3, 4, 5, 6)] + [
    (40, 8, 0, 61, 1, False), (25, 17, 8, 62, 2, False), (65, 230, 8, 83, 3, False),
    (60, 45, 9, 84, 2, True), (60, 45, 36, 81, 1, True), (60, 45, 41, 82, 1, True)]


@pytest.mark.parametrize("nz,nx,nb,nt,nshots,fs", CASES)
def test_four_steps_agree_with_two_and_oracle(nz, nx, nb, nt, nshots, fs):
    print(f"case: four steps {nz}x{nx} nb{nb} nt{nt} {nshots} shots fs{fs}", file=sys.stderr, flush=True)
    nh = 3
    w = synth.tiny(nz=nz, nx=nx, nb=nb, nt=nt, nshots=nshots, nh=nh, seed=21)
    w.rec_ix[:, -1] = w.rec_ix[:, 0]            # two receivers in one cell
    g, geo, vel = oracle_problem_f32(w)
    grid, tv, tg = gpu_problem(w)
    g.free_surface = grid.free_surface = fs
    pt = _dev(0.2 * synth.random_ptilde(nh, nz, nx, 3))
    data = _dev(np.random.default_rng(4).standard_normal((nshots, w.nrec, nt)))
    dobs = _dev(0.7 * oracle.model(g, vel, geo))
    dso = synth.dso_weights(nh)
    got = []
    for steps in (2, 4):
        ctx = _ctx(steps)
        got.append([_np(t) for t in (ctx.model(grid, tv, tg), *ctx.gradient(grid, tv, tg, pt, dobs, 1e-3, dso),
                                     ctx.born_ext_fwd(grid, tv, tg, pt), ctx.born_ext_adj(grid, tv, tg, data, nh))])
        ctx.close()
    for a, b in zip(got[0][:4], got[1][:4]):
        assert np.array_equal(a, b)
    for a, b in zip(got[0][4:], got[1][4:]):
        assert np.linalg.norm(a - b) <= 1e-7 * np.linalg.norm(a)
    ref = [oracle.model(g, vel, geo), *oracle.gradient(g, vel, geo, _np(pt), _np(dobs), 1e-3, dso)[1:],
           oracle.born_ext_fwd(g, vel, geo, _np(pt)), oracle.born_ext_adj(g, vel, geo, _np(data), nh)]
    for a, b in zip([got[1][0]] + got[1][2:], ref):
        assert np.linalg.norm(a - b) <= 1e-4 * np.linalg.norm(b)
