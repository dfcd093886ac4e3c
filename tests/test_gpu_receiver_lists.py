"""Receiver injection lists of the two-step kernel against the oracle.

A wavefront's list goes through LDS when its cells are all different and entry
by entry when one repeats; lists longer than 64 entries take several batches.
The adjoint (receivers as sources) and the modeled data of layouts that reach
each branch match the oracle at the suite's 1e-4.
"""
import sys

import numpy as np
import pytest

import oracle
import synth
from _helpers import gpu_problem, oracle_problem_f32, rel_l2

pytestmark = pytest.mark.gpu


def _layout(kind, nz, nx):
    if kind == "line":                      # one receiver a column
        return np.full(nx, 3), np.arange(nx)
    if kind == "repeats":                   # every cell twice, out of order, one three times
        ix = np.concatenate([np.arange(nx)[::-1], np.arange(nx), [5]])
        return np.full(ix.size, 3), ix
    if kind == "block":                     # more than 64 different cells for one wavefront
        iz, ix = np.meshgrid(np.arange(nz), np.arange(10, 16))
        return iz.ravel(), ix.ravel()
    iz, ix = np.meshgrid(np.arange(nz), np.arange(10, 13))   # the same, with repeats
    return np.tile(iz.ravel(), 2), np.tile(ix.ravel(), 2)


@pytest.mark.parametrize("kind", ["line", "repeats", "block", "block-repeats"])
def test_receiver_layouts_match_oracle(kind):
    import torch
    import paper_2206_02362_amd as fw
    print(f"case: receiver lists {kind}, 60x45", file=sys.stderr, flush=True)
    nz, nx = 60, 45
    w = synth.tiny(nz=nz, nx=nx, nb=7, nt=141, nshots=2, nh=3, seed=8)
    iz, ix = _layout(kind, nz, nx)
    w.rec_iz = np.tile(iz, (2, 1)).astype(np.int32)
    w.rec_ix = np.tile(ix, (2, 1)).astype(np.int32)
    g, geo, vel = oracle_problem_f32(w)
    grid, tv, tg = gpu_problem(w)
    data = np.random.default_rng(2).standard_normal((2, ix.size, w.nt)).astype(np.float32)
    ctx = fw.Context(0)
    img = ctx.born_ext_adj(grid, tv, tg, torch.tensor(data, device="cuda:0"), 3).double().cpu().numpy()
    mod = ctx.model(grid, tv, tg).double().cpu().numpy()
    ctx.close()
    assert rel_l2(img, oracle.born_ext_adj(g, vel, geo, data.astype(np.float64), 3)) < 1e-4
    assert rel_l2(mod, oracle.model(g, vel, geo)) < 1e-4
