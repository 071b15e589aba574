"""The one-map kernel's product basis of the harmonics at every m_max, against direct trigonometry
in the oracle; bearings packed at 0 and pi, where a basis that cancels would lose digits."""

import math

import numpy as np
import pytest

from synth.bins import chord2_edges, theta_edges
from tests import gpu_helpers as G

pytestmark = pytest.mark.gpu


def _meridian(n, rng):
    """Points within 1e-3 deg of one meridian: every bearing is close to 0 or pi."""
    lat = np.radians(rng.uniform(10.0, 20.0, n))
    lon = np.radians(rng.uniform(-1e-3, 1e-3, n))
    return np.stack([np.cos(lat) * np.cos(lon), np.cos(lat) * np.sin(lon), np.sin(lat)])


def _cap(n, rng):
    lat = np.radians(rng.uniform(-35.0, -28.0, n))
    lon = np.radians(rng.uniform(40.0, 48.0, n))
    return np.stack([np.cos(lat) * np.cos(lon), np.cos(lat) * np.sin(lon), np.sin(lat)])


@pytest.mark.parametrize("m_max", list(range(17)))
@pytest.mark.parametrize("points", [_meridian, _cap])
def test_harmonics_of_every_degree(points, m_max):
    G.say("case: harmonics", points.__name__, m_max)
    rng = np.random.default_rng(100 + m_max)
    n = 300
    xyz = points(n, rng)
    x = rng.normal(size=n)
    E = chord2_edges(theta_edges(math.radians(0.3), math.radians(6.0), 3, False))
    idx = G.build(xyz, x, E)
    pm = G.perm(idx)
    a, W, N, _ = G.gpu_multipoles(idx, m_max, 0, n, norm="none")
    ao, Wo, No, _, _ = G.oracle_multipoles(xyz, x, np.ones(n), E, m_max, pm)
    assert np.array_equal(N, No) and np.array_equal(W, Wo)
    # sum |v| of each (pivot, bin): the m = 0 sums of |x|
    absum, *_ = G.oracle_multipoles(xyz, np.abs(x), np.ones(n), E, 0, pm)
    # the bearing is good to ~2e-14 rad (one Newton step from an FP32 seed), which degree m
    # multiplies by m <= 16; up to 300 rounded additions, through up to 8 sums of the
    # recovery, add 300 x 8 x 1.1e-16: together below 1e-12 of sum |v|
    assert np.all(np.abs(a - ao) <= 1e-12 * absum.real + 1e-300)
