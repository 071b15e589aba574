"""The one-map kernel over window lists against the same kernel band by band: a request for
neighbour fingerprints takes the second, anything else at these sizes the first.  Both visit
the same pairs in the same order, so every output agrees to the last bit."""

import math

import numpy as np
import pytest
import torch

import paper_2408_16847_amd as z3
from synth import cap_points, plane_points, ring_centres
from synth.bins import chord2_edges, theta_edges
from tests import gpu_helpers as G

pytestmark = pytest.mark.gpu

DEG = math.pi / 180.0


def _check(idx, m_max, prec, ranges):
    for p0, p1 in ranges:
        lists = z3.accumulate(idx, m_max, p0, p1, prec=prec, want_w=True, want_counts=True)
        bands = z3.accumulate(idx, m_max, p0, p1, prec=prec, want_w=True, want_counts=True, want_idhash=True)
        for k in ("A", "W", "counts"):
            assert torch.equal(lists[k], bands[k]), (k, p0, p1)


@pytest.mark.parametrize("prec,m_max", [("fp64", 0), ("fp64", 10), ("mixed", 16)])
@pytest.mark.parametrize("cell", [0.0, 0.002, 0.03, 0.7])
def test_sky(prec, m_max, cell):
    # band heights from a fifth of a bin (many lists per bin) to one band for everything; a cap
    # that wraps through longitude 0, with weights
    G.say("case: window lists, cap", prec, m_max, cell)
    xyz = cap_points(3000, 10.0, seed=8).numpy()
    rng = np.random.default_rng(9)
    E = chord2_edges(theta_edges(0.3 * DEG, 4.0 * DEG, 6, True))
    idx = G.build(xyz, rng.normal(size=3000), E, w=rng.uniform(0.5, 2.0, 3000), cell_size=cell)
    _check(idx, m_max, prec, [(0, 3000), (1, 2), (1700, 1999)])


def test_poles_and_full_circles():
    # pivots on both sides of the poles, windows that cover whole bands, empty bands between
    G.say("case: window lists, poles")
    ring = ring_centres(16).numpy()
    keep = np.abs(ring[2]) > 0.8
    xyz = np.ascontiguousarray(ring[:, keep])
    rng = np.random.default_rng(10)
    n = xyz.shape[1]
    E = chord2_edges(theta_edges(2.0 * DEG, 179.0 * DEG, 9, False))
    idx = G.build(xyz, rng.normal(size=n), E, cell_size=0.01)
    _check(idx, 7, "fp64", [(0, n), (n - 65, n)])


def test_plane():
    G.say("case: window lists, plane")
    xy = plane_points(40, seed=2)
    E = np.linspace(0.8, 7.0, 8) ** 2
    for cell in (0.0, 0.3, 100.0):
        idx = z3.Index(xy.cuda(), E, cell_size=cell, planar=True)
        idx.set_values(torch.randn(xy.shape[1], dtype=torch.float64, device="cuda"))
        _check(idx, 9, "fp64", [(0, xy.shape[1])])
