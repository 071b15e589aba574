"""The MFMA kernel that lays many bins end to end: bins of few pairs in every block shape, against
one-map estimates, and the rule that chooses it against the kernel of one bin at a time."""

import math

import numpy as np
import pytest
import torch

import paper_2408_16847_amd as z3
from synth import cap_points
from synth.bins import chord2_edges, theta_edges
from tests import gpu_helpers as G

pytestmark = pytest.mark.gpu


# 64 bins fill the run table; the first bins hold few or no pairs.
@pytest.mark.parametrize("n", [900, 5000])
@pytest.mark.parametrize("shape", [(4, 16), (2, 32), (2, 16), (4, 32)])
@pytest.mark.parametrize("nbins,cell,m_max", [(1, 0.0, 0), (7, 0.0, 7), (64, 0.0, 3), (6, 0.02, 16)])
def test_bins_end_to_end_equal_single_maps(n, shape, nbins, cell, m_max):
    G.say("case: batch bins", n, shape, nbins, cell, m_max)
    xyz = cap_points(n, 10.0, seed=31).numpy()
    rng = np.random.default_rng(32)
    nmaps = 37
    x = rng.normal(size=(nmaps, n))
    w = rng.uniform(0.5, 2.0, n)
    E = chord2_edges(theta_edges(math.radians(0.1), math.radians(2.5), nbins, True))
    idx = G.build(xyz, x, E, w=w, cell_size=cell)
    idx.set_batch_shape(*shape)
    z, pairs = z3.estimate_maps(idx, m_max)
    for k in (0, 15, 16, 36):
        zk, pk = z3.estimate(idx, m_max, map_index=k)
        assert pk == pairs
        # two orders of the same sums, harmonics good to ~4e-13 at m = 16
        assert G.err_m(z[k], zk).max() < 1e-11
    idx.free()


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("shape", [(4, 16), (2, 32), (2, 16), (4, 32)])
@pytest.mark.parametrize("nbins,cell,m_max", [(1, 0.4, 0), (9, 0.4, 10), (40, 0.05, 16)])
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_both_kernels_sum_alike(weighted, shape, nbins, cell, m_max, prec):
    """Bins of up to 360 bands (several runs a bin, more windows than a block has threads) and of
    few.  A polar cap of 100 and more pairs a bin, and the same cap with one point at the other pole,
    far from every pivot, which lowers the mean density below the rule's line.  The cell size (degrees) is given: an
    automatic one follows the density, and with it the order of the candidates."""
    G.say("case: both batch kernels", weighted, shape, nbins, cell, m_max, prec)
    n, nmaps = 5000, 37
    cap = cap_points(n, 10.0, seed=33).numpy()[[1, 2, 0]]
    far = np.array([[0.0], [0.0], [-1.0]])
    rng = np.random.default_rng(34)
    x = rng.normal(size=(nmaps, n))
    w = rng.uniform(0.5, 2.0, n) if weighted else np.ones(n)
    E = chord2_edges(theta_edges(math.radians(0.1), math.radians(9.0), nbins, False))
    sums = []
    for xyz, xs, ws in ((cap, x, w), (np.hstack([cap, far]), np.hstack([x, x[:, :1]]), np.append(w, 1.0))):
        idx = G.build(xyz, xs, E, w=ws if weighted else None, cell_size=math.radians(cell))
        idx.set_batch_shape(*shape)
        zeta = torch.zeros((nmaps, m_max + 1, nbins, nbins, 2), dtype=torch.float64, device="cuda")
        pairs = torch.zeros(1, dtype=torch.int64, device="cuda")
        z3.estimate_maps_raw(idx, m_max, prec, 0, n, zeta, pairs)
        sums.append((zeta.cpu().numpy(), int(pairs.item())))
        idx.free()
    (za, pa), (zb, pb) = sums
    assert pa == pb
    # the same sums in the same order; only the pivots' order can differ, in FP64: terms of order
    # 1 (multipoles are means of unit-variance values), 5,000 pivots
    assert np.abs(za - zb).max() < 5000 * 1e-12
