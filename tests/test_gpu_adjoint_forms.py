"""The adjoint's scatter in each of its forms (four, two or one map per lane; a window's segments
joined or one after the other) against the oracle gradient."""

import math

import numpy as np
import pytest
import torch

import paper_2408_16847_amd as z3
from oracle import grad as ograd
from oracle import ref as oref
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


def _pivot_grad(xyz, w, x, edges, m_max, Gc, piv, planar):
    """Gradient of sum over the pivots `piv` alone of v_p X_p X_p^H, from the definition."""
    nb = len(edges) - 1
    raw = oref.multipoles_planar if planar else oref.multipoles
    a, W, _ = raw(xyz[:, piv], xyz, w, x, edges, m_max)
    X = oref.normalise(a, W)
    grad = np.zeros(xyz.shape[1])
    for m in range(m_max + 1):
        grad[piv] += w[piv] * np.einsum("pa,ab,pb->p", X[:, m], np.conj(Gc[m]), np.conj(X[:, m])).real
    D = np.einsum("mab,pmb->pma", np.conj(Gc) + np.swapaxes(Gc, 1, 2), np.conj(X))
    if not planar:
        north, east = oref.bearing_basis(xyz[:, piv])
    for i, p in enumerate(piv):
        d = xyz - xyz[:, p:p + 1]
        d2 = d[0] * d[0] + d[1] * d[1] if planar else (d[0] * d[0] + d[1] * d[1]) + d[2] * d[2]
        b = oref.bin_index(d2, edges)
        js = np.nonzero(b >= 0)[0]
        d = d[:, js]
        phi = oref.planar_bearing(d[0], d[1]) if planar else oref.bearing(d, north[:, i:i + 1], east[:, i:i + 1])
        tot = np.zeros(js.size)
        for m in range(m_max + 1):
            tot += (np.exp(-1j * m * phi) * D[i, m, b[js]]).real
        np.add.at(grad, js, w[p] * x[p] * w[js] / W[i, b[js]] * tot)
    return grad


# One map, bands so tall that the records a wave's windows reach do not fit the LDS slice (1,024): their
# contributions go to memory one by one.  Few pairs by the mean density: the two segments joined;
# many: one after the other.
@pytest.mark.parametrize("planar", [False, True])
@pytest.mark.parametrize("joined", [False, True])
def test_spans_wider_than_the_lds_slice(planar, joined):
    G.say("case: adjoint spans", planar, joined)
    rng = np.random.default_rng(61)
    m_max = 3
    if planar:
        n = 16000
        xyz = rng.uniform(0.0, 100.0, (2, n))
        E = np.linspace(0.5, 3.5 if joined else 12.0, 7) ** 2
        cell = 200.0
        reads = n / 1e4 * math.pi * (E[-1] - E[0])
    else:
        n = 6000
        xyz = cap_points(n, 5.0, seed=62).numpy()
        E = chord2_edges(theta_edges(math.radians(0.2), math.radians(1.5 if joined else 6.0), 6, False))
        cell = 0.4
        th = np.arctan2(np.hypot(xyz[0], xyz[1]), xyz[2])
        reads = n / (2.0 * math.pi * (math.cos(th.min()) - math.cos(th.max()))) * math.pi * (E[-1] - E[0])
    # the rule's windows: the bins' diameters in bands, two a band, and two more
    radii = np.sqrt(E[1:]) if planar else 2.0 * np.arcsin(np.sqrt(E[1:]) / 2.0)
    assert (reads < 8.0 * (4.0 * radii / cell + 2.0).sum()) == joined
    x = rng.normal(size=n)
    w = rng.uniform(0.5, 2.0, n)
    Gc = rng.normal(size=(m_max + 1, 6, 6)) + 1j * rng.normal(size=(m_max + 1, 6, 6))
    Gt = torch.from_numpy(np.stack([Gc.real, Gc.imag], -1)).cuda()
    idx = z3.Index(torch.from_numpy(xyz).cuda(), E, weights=torch.from_numpy(w).cuda(), cell_size=cell, planar=planar)
    idx.set_values(torch.from_numpy(x).cuda())
    p0, p1 = 1001, 1140  # two whole waves and a part of one
    piv = G.perm(idx)[p0:p1]
    # the premise: in the one band, consecutive index points are neighbours along it, and a wave's widest
    # window alone reaches more records than the slice holds
    along = xyz[0] if planar else np.arctan2(xyz[1], xyz[0])
    reach = radii[-1] * 0.95
    assert ((along > along[piv[70]] - reach) & (along < along[piv[70]] + reach)).sum() > 1024
    got = z3.adjoint(idx, Gt, 1.0, m_max, p0=p0, p1=p1).cpu().numpy()
    ref = _pivot_grad(xyz, w, x, E, m_max, Gc, piv, planar)
    # FP64 sums of at most 139 pivots and 6,000 neighbours, in any order
    assert np.abs(got - ref).max() < 1e-11 * np.abs(ref).max()
    idx.free()
