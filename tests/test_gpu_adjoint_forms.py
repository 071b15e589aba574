"""The adjoint's scatter in each of its forms (four, two or one map per lane; a window's segments
joined or one after the other) against the oracle gradient."""

import math

import numpy as np
import pytest
import torch

import paper_2408_16847_amd as z3
from oracle import grad as ograd
from synth import cap_points
from synth.bins import chord2_edges, theta_edges
from tests import gpu_helpers as G

pytestmark = pytest.mark.gpu


# a cell size of 0.35 rad puts the cap in one band of long windows, 0.0 gives short ones.  The polar cap
# holds the first band (records from 0 on) and windows with an empty second segment.
@pytest.mark.parametrize("m_max", [0, 9, 10, 11, 12, 16])
@pytest.mark.parametrize("nmaps", [1, 2, 3, 7])
@pytest.mark.parametrize("cell", [0.0, 0.35])
@pytest.mark.parametrize("polar", [False, True])
def test_every_form_matches_oracle(m_max, nmaps, cell, polar):
    G.say("case: adjoint forms", m_max, nmaps, cell, polar)
    n, nbins = 400, 4
    xyz = cap_points(n, 8.0, seed=51).numpy()
    if polar:
        xyz = np.ascontiguousarray(xyz[[1, 2, 0]])
    rng = np.random.default_rng(52)
    x = rng.normal(size=(nmaps, n))
    w = rng.uniform(0.5, 2.0, n)
    E = chord2_edges(theta_edges(math.radians(0.3), math.radians(4.0), nbins, True))
    Gc = rng.normal(size=(nmaps, m_max + 1, nbins, nbins)) + 1j * rng.normal(size=(nmaps, m_max + 1, nbins, nbins))
    Gt = torch.from_numpy(np.stack([Gc.real, Gc.imag], -1)).cuda()
    idx = G.build(xyz, x, E, w=w, cell_size=cell)
    got = z3.adjoint_maps(idx, Gt, 1.0 / w.sum(), m_max).cpu().numpy().reshape(nmaps, n)
    for k in sorted({0, nmaps - 1}):
        ref = ograd.zeta_grad(xyz, w, x[k], E, m_max, Gc[k])
        one = z3.adjoint(idx, Gt[k], 1.0 / w.sum(), m_max, map_index=k).cpu().numpy()
        # FP64 sums of at most 400 pivots in any order, harmonics good to ~4e-13 at m = 16
        assert np.abs(got[k] - ref).max() < 1e-11 * np.abs(ref).max()
        assert np.abs(one - ref).max() < 1e-11 * np.abs(ref).max()
    idx.free()
