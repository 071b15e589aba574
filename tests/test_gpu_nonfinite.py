"""Values that are not finite: they reach the sums of the bins that hold them and, where several maps go
together, no other map.  Every kernel form is compared with the same form on finite values."""

import math

import numpy as np
import pytest
import torch

import paper_2408_16847_amd as z3
from synth import cap_points, plane_points
from synth.bins import chord2_edges, theta_edges
from tests import gpu_helpers as G

pytestmark = pytest.mark.gpu

N, BAD = 1500, (3, 700, 1499)
VALUES = [math.nan, math.inf, -math.inf]


def _catalogue():
    xyz = cap_points(N, 9.0, seed=71).numpy()
    E = chord2_edges(theta_edges(math.radians(0.4), math.radians(3.0), 4, True))
    return xyz, E


def _spoil(x, bad):
    y = x.copy()
    y[..., list(BAD)] = bad
    return y


@pytest.mark.parametrize("bad", VALUES)
@pytest.mark.parametrize("planar", [False, True])
@pytest.mark.parametrize("cell", [0.0, 0.5])  # short windows (lists) and one tall band
def test_one_map(bad, planar, cell):
    G.say("case: not finite, one map", bad, planar, cell)
    rng = np.random.default_rng(72)
    if planar:
        pos, E = plane_points(40, seed=3).numpy()[:, :N], np.linspace(0.8, 5.0, 5) ** 2
        cell *= 50.0
    else:
        pos, E = _catalogue()
    x = rng.normal(size=N)
    out = []
    for val in (x, _spoil(x, bad), _spoil(np.zeros(N), 1.0)):
        idx = z3.Index(torch.from_numpy(np.ascontiguousarray(pos)).cuda(), E, cell_size=cell, planar=planar)
        idx.set_values(torch.from_numpy(val).cuda())
        out.append(z3.accumulate(idx, 6, want_w=True, want_counts=True))
        idx.free()
    clean, spoilt, where = out
    hit = where["A"][0, 0] != 0.0  # bins that hold a bad point
    assert bool(hit.any()) and not bool(hit.all())
    assert torch.equal(clean["W"], spoilt["W"]) and torch.equal(clean["counts"], spoilt["counts"])
    assert torch.equal(clean["A"][:, :, ~hit], spoilt["A"][:, :, ~hit])
    assert not bool(torch.isfinite(spoilt["A"][0, 0][hit]).any())


# three and four maps a lane, two at a time (m_max 12), and the matrix-core kernel: bins of few pairs
# end to end, or (a tall band and many points a bin) one at a time
@pytest.mark.parametrize("bad", VALUES)
@pytest.mark.parametrize("nmaps,m_max,shape", [(3, 5, None), (4, 5, None), (4, 12, None), (7, 5, (2, 16)), (40, 3, (4, 16))])
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("cell", [0.0, 0.5])
def test_other_maps_are_untouched(bad, nmaps, m_max, shape, prec, cell):
    G.say("case: not finite, maps", bad, nmaps, m_max, prec, cell)
    xyz, E = _catalogue()
    x = np.random.default_rng(73).normal(size=(nmaps, N))
    y = x.copy()
    y[1] = _spoil(x[1], bad)
    out = []
    for val in (x, y):
        idx = G.build(xyz, val, E, cell_size=cell)
        if shape:
            idx.set_batch_shape(*shape)
        out.append(z3.estimate_maps(idx, m_max, prec=prec))
        idx.free()
    (clean, pairs), (spoilt, pairs2) = out
    others = [k for k in range(nmaps) if k != 1]
    assert pairs == pairs2
    assert np.array_equal(clean[others], spoilt[others])
    assert not np.isfinite(spoilt[1][0]).any()


@pytest.mark.parametrize("bad", VALUES)
@pytest.mark.parametrize("nmaps,cell", [(1, 0.0), (1, 0.5), (4, 0.0)])
def test_adjoint(bad, nmaps, cell):
    # a pivot's bad value reaches its neighbours and itself, a neighbour's the pivots around it and theirs:
    # points further away than two bins keep their gradient
    G.say("case: not finite, adjoint", bad, nmaps, cell)
    xyz, E = _catalogue()
    rng = np.random.default_rng(74)
    x = rng.normal(size=(nmaps, N))
    y = x.copy()
    y[0, BAD[0]] = bad
    Gt = torch.from_numpy(rng.normal(size=(nmaps, 6, 4, 4, 2))).cuda()
    out = []
    for val in (x, y):
        idx = G.build(xyz, val, E, cell_size=cell)
        out.append(z3.adjoint_maps(idx, Gt, 1.0, 5).cpu().numpy())
        idx.free()
    clean, spoilt = out
    far = ((xyz - xyz[:, BAD[0]:BAD[0] + 1]) ** 2).sum(0) > (2.0 * math.sqrt(E[-1])) ** 2
    near = ((xyz - xyz[:, BAD[0]:BAD[0] + 1]) ** 2).sum(0) < E[-1]
    scale = np.abs(clean).max()
    assert far.sum() > 100 and np.abs(spoilt[0][far] - clean[0][far]).max() <= 1e-12 * scale
    assert np.abs(spoilt[1:] - clean[1:]).max(initial=0.0) <= 1e-12 * scale
    assert not np.isfinite(spoilt[0][near]).all()


@pytest.mark.parametrize("bad", VALUES)
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("nbins", [3, 8, 9, 20, 33])
def test_contraction(bad, prec, nbins):
    # one bin of one pivot, in the middle and in the ragged end of the pivots
    G.say("case: not finite, contraction", bad, prec, nbins)
    g = torch.Generator(device="cuda").manual_seed(nbins)
    P, M = 1003, 2
    A = torch.randn((M + 1, 2, nbins, P), dtype=torch.float64, device="cuda", generator=g)
    A = A if prec == "fp64" else A.float()
    v = torch.randn(P, dtype=torch.float64, device="cuda", generator=g)
    for p in (517, P - 1):
        B = A.clone()
        B[1, 0, nbins - 1, p] = bad
        clean, spoilt = z3.contract(A, v, M, nbins, prec), z3.contract(B, v, M, nbins, prec)
        assert torch.equal(clean[[0, 2]], spoilt[[0, 2]])
        assert torch.equal(clean[1, :-1, :-1], spoilt[1, :-1, :-1])
        assert not bool(torch.isfinite(spoilt[1, -1, :-1, 0]).any())
