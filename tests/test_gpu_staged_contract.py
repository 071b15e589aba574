"""The contraction of the many-map kernel's staging at the edges of its loads and tiles: the largest
m_max of each number of row tiles, bins on both sides of a tile, and pivot ranges around a tile of
16, against one-map estimates of the same pivots."""

import math

import numpy as np
import pytest
import torch

import paper_2408_16847_amd as z3
from synth import cap_points
from synth.bins import chord2_edges, theta_edges
from tests import gpu_helpers as G

pytestmark = pytest.mark.gpu


def _raw(idx, m_max, prec, p0, p1):
    zeta = torch.zeros((idx.nmaps, m_max + 1, idx.nbins, idx.nbins, 2), dtype=torch.float64, device="cuda")
    z3.estimate_maps_raw(idx, m_max, prec, p0, p1, zeta, None)
    return zeta.cpu().numpy()


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("nbins,m_max", [(1, 0), (1, 16), (8, 16), (9, 12), (16, 12), (16, 16), (17, 4), (24, 5), (24, 11),
                                         (25, 6), (32, 6), (40, 3), (64, 1)])
@pytest.mark.parametrize("p0,p1", [(5, 6), (0, 15), (3, 19), (10, 27), (0, 300)])
def test_staged_contraction_edges(prec, nbins, m_max, p0, p1):
    G.say("case: staged contraction", prec, nbins, m_max, p0, p1)
    n, nmaps = 300, 5
    xyz = cap_points(n, 4.0, seed=41).numpy()
    x = np.random.default_rng(42).uniform(0.0, 1.0, (nmaps, n))
    E = chord2_edges(theta_edges(math.radians(0.2), math.radians(8.0), nbins, False))
    idx = G.build(xyz, x, E)
    idx.set_batch_shape(2, 16)
    z = _raw(idx, m_max, prec, p0, p1)
    idx.free()
    for k in (0, 4):
        one = G.build(xyz, x[k : k + 1], E)
        zk = _raw(one, m_max, "fp64", p0, p1)[0]
        one.free()
        # |x| <= 1, so is every multipole: the terms of an entry sum to at most the pivots.  FP64:
        # 300 terms through harmonics good to 4e-13; mixed: 66 roundings of 6e-8 in the contraction
        # and 40 in each multipole
        tol = (p1 - p0) * (1e-12 if prec == "fp64" else 146 * 6e-8)
        assert np.abs(z[k] - zk).max() <= tol
