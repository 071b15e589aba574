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


@pytest.mark.parametrize("lo,hi,nb", [(1.5, 8.0, 10), (3.0, 20.0, 6), (12.0, 30.0, 2)])
@pytest.mark.parametrize("radius", [12.0, 40.0])
def test_pixelised_patch(lo, hi, nb, radius):
    # a patch's density over its colatitude range reads low: real windows of 3 to 70 pairs, which the rule
    # reads as 0.5 to 30, so that these cases lie on both sides of its line
    G.say("case: window lists, patch", lo, hi, nb, radius)
    ring = ring_centres(48).numpy()
    centre = np.array([math.cos(0.5), 0.0, math.sin(0.5)])
    xyz = np.ascontiguousarray(ring[:, centre @ ring > math.cos(radius * DEG)])
    n, pixel = xyz.shape[1], 60.0 / 48 * DEG
    x = np.random.default_rng(11).normal(size=n)
    E = chord2_edges(theta_edges(lo * pixel, hi * pixel, nb, True))
    idx = G.build(xyz, x, E)
    _check(idx, 8, "fp64", [(0, n), (n // 2, n // 2 + 70)])
    p0 = n // 3
    a, W, N, H = G.gpu_multipoles(idx, 8, p0, p0 + 40, norm="none")
    lists = z3.accumulate(idx, 8, p0, p0 + 40, norm="none", want_counts=True)
    ao, Wo, No, _, Ho = G.oracle_multipoles(xyz, x, np.ones(n), E, 8, G.perm(idx)[p0:p0 + 40])
    assert np.array_equal(N, No) and np.array_equal(H, Ho)
    assert np.array_equal(lists["counts"].cpu().numpy().T, No)
    A = lists["A"].cpu().numpy()
    got = np.transpose(A[:, 0] + 1j * A[:, 1], (2, 0, 1))
    # sums of at most 2,500 values of size one, harmonics good to ~1e-14
    assert np.abs(got - ao).max() < 1e-10
    idx.free()
