"""Launches of few pivot blocks split their radial bins over the grid: every bin must be
visited exactly once, whatever the number of bins, their widths and the number of groups."""

import math

import numpy as np
import pytest
import torch

import paper_2408_16847_amd as z3
from synth import cap_points
from synth.bins import chord2_edges, theta_edges
from tests import gpu_helpers as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nbins,log", [(1, False), (2, True), (13, False), (64, True), (64, False)])
def test_one_group_per_bin(nbins, log):
    G.say("case: bin groups", nbins, log)
    xyz = cap_points(700, 10.0, seed=3).numpy()
    x = np.random.default_rng(5).normal(size=700)
    E = chord2_edges(theta_edges(math.radians(0.2), math.radians(3.0), nbins, log))
    idx = G.build(xyz, x, E)
    pm = G.perm(idx)
    a, W, N, H = G.gpu_multipoles(idx, 5, 0, 700, norm="none")
    ao, Wo, No, _, Ho = G.oracle_multipoles(xyz, x, np.ones(700), E, 5, pm)
    assert np.array_equal(N, No) and np.array_equal(W, Wo) and np.array_equal(H, Ho)
    # the bar of the per-pivot multipoles: 1e-11 of each (pivot, bin)'s scale
    assert (np.abs(a - ao) / (np.abs(ao).max(axis=1, keepdims=True) + 1e-300)).max() < 1e-11


@pytest.mark.parametrize("n,nbins", [(33_100, 64), (100_000, 64), (190_001, 20)])
def test_several_bins_per_group(n, nbins):
    # the whole range takes 63, 21 and 12 groups; a short range takes one group per bin, which
    # the test above holds against the oracle
    G.say("case: several bins per group", n, nbins)
    xyz = cap_points(n, 10.0, seed=4)
    x = np.random.default_rng(6).normal(size=n)
    E = chord2_edges(theta_edges(math.radians(0.05), math.radians(0.6), nbins, True))
    idx = G.build(xyz.numpy(), x, E)
    whole = z3.accumulate(idx, 4, want_w=True, want_counts=True, want_idhash=True)
    for p0, p1 in ((0, 700), (n // 2 + 11, n // 2 + 800), (n - 513, n)):
        part = z3.accumulate(idx, 4, p0, p1, want_w=True, want_counts=True, want_idhash=True)
        for k in ("A", "W", "counts", "idhash"):
            assert torch.equal(whole[k][..., p0:p1], part[k]), k
