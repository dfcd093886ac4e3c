"""Extended-precision fields: the same bits from both multi-step kernels.

The Born pair, the variable-projection step and the time-lag pair carry their
background in FP32 + BF16 with an update in FP64.  Its arithmetic is spelled out
once for the two-step and the four-step kernel, so results do not depend on
which of them a call's size selects: with either kernel forced, and for a shot
alone (four steps per launch) against the same shot in a set (two).
"""
import os
import sys

import numpy as np
import pytest

import synth
from _helpers import gpu_problem

pytestmark = pytest.mark.gpu


def _ctx(steps=None):
    import paper_2206_02362_amd as fw
    if steps:
        os.environ["FWIME_STEPS"] = str(steps)
    try:
        return fw.Context(0)
    finally:
        os.environ.pop("FWIME_STEPS", None)


def _dev(a):
    import torch
    return torch.tensor(np.asarray(a), dtype=torch.float32, device="cuda:0")


@pytest.mark.parametrize("nz,nx,nb,nt,nshots,fs", [(25, 17, 8, 62, 2, False), (65, 230, 8, 83, 3, False),
                                                   (60, 45, 36, 81, 1, True), (100, 200, 40, 1000, 2, False)])
def test_two_and_four_steps_agree_bit_for_bit(nz, nx, nb, nt, nshots, fs):
    import torch
    print(f"case: extended precision, 2 against 4 steps {nz}x{nx} nb{nb} nt{nt} fs{fs}", file=sys.stderr, flush=True)
    w = synth.tiny(nz=nz, nx=nx, nb=nb, nt=nt, nshots=nshots, nh=5, seed=31)
    grid, tv, tg = gpu_problem(w)
    grid.free_surface = fs
    pt = _dev(0.2 * synth.random_ptilde(5, nz, nx, 3))
    data = _dev(np.random.default_rng(4).standard_normal((nshots, w.nrec, nt)))
    got = []
    for steps in (2, 4):
        ctx = _ctx(steps)
        p, phi = ctx.vp_solve(grid, tv, tg, data, 5, 1e-3, synth.dso_weights(5), 2)
        got.append([ctx.born_ext_fwd(grid, tv, tg, pt), ctx.born_ext_adj(grid, tv, tg, data, 5), p, torch.as_tensor(phi),
                    ctx.born_ext_tau_fwd(grid, tv, tg, pt, 3), ctx.born_ext_tau_adj(grid, tv, tg, data, 5, 3)])
        ctx.close()
    for a, b in zip(*got):
        assert torch.equal(a, b)


def test_born_shot_alone_and_in_a_set():
    import torch
    import paper_2206_02362_amd as fw
    n = 8                                       # 27 two-step workgroups a shot: 216, above the limit of 160
    w = synth.tiny(nz=100, nx=200, nb=30, nt=1000, nshots=n, nh=5, seed=32)
    grid, tv, tg = gpu_problem(w)
    pt = _dev(0.2 * synth.random_ptilde(5, 100, 200, 3))
    ctx = _ctx()
    both = ctx.born_ext_fwd(grid, tv, tg, pt)
    for s in (0, n - 1):
        one = fw.Geometry(w.src_iz[s:s + 1], w.src_ix[s:s + 1], w.rec_iz[s:s + 1], w.rec_ix[s:s + 1],
                          tg.wavelet[s:s + 1].contiguous())
        assert torch.equal(ctx.born_ext_fwd(grid, tv, one, pt)[0], both[s])
    ctx.close()
