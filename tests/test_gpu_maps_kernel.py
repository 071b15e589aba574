"""The register-tiled many-map kernel at the edges of its variants (three maps a lane, four, or
two at a time; requests ahead or not; window lists or bands in lockstep) against one-map
estimates of the same maps."""

import math

import numpy as np
import pytest

import paper_2408_16847_amd as z3
from synth import cap_points
from synth.bins import chord2_edges, theta_edges
from tests import gpu_helpers as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m_max", [0, 6, 7, 10, 11, 12, 13, 14, 15, 16])
@pytest.mark.parametrize("nmaps", [3, 4])
@pytest.mark.parametrize("cell", [0.0, 0.3])  # short windows (lists) and long ones
def test_group_equals_single_maps(m_max, nmaps, cell):
    G.say("case: maps kernel", m_max, nmaps, cell)
    n = 900
    xyz = cap_points(n, 10.0, seed=21).numpy()
    rng = np.random.default_rng(22)
    x = rng.normal(size=(nmaps, n))
    w = rng.uniform(0.5, 2.0, n)
    E = chord2_edges(theta_edges(math.radians(0.5), math.radians(5.0), 4, True))
    idx = G.build(xyz, x, E, w=w, cell_size=cell)
    z, pairs = z3.estimate_maps(idx, m_max)
    for k in range(nmaps):
        zk, pk = z3.estimate(idx, m_max, map_index=k)
        assert pk == pairs
        # two orders of the same sums (at most 900 terms, products of two), through harmonics
        # that are good to ~4e-13 at m = 16: below 1e-11 of each m's largest entry
        assert G.err_m(z[k], zk).max() < 1e-11
