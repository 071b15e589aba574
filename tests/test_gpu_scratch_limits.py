"""The contraction's partial sums where there is little room for them: under an allocation limit, and
in a capture's reservation.  A call that fits with one partial sum per 4,096 pivots runs, with the
same result up to the order of the sums."""

import ctypes

import numpy as np
import pytest
import torch

import paper_2408_16847_amd as z3
from paper_2408_16847_amd import _lib
from synth import cap_points
from synth.bins import arcmin, chord2_edges, theta_edges
from tests import gpu_helpers as G

pytestmark = pytest.mark.gpu

SIZE_MAX = ctypes.c_size_t(-1).value


def _least(npiv, m_max, nbins, maps=1, cross=False):
    """Bytes of one 2 KiB partial sum per 4,096 pivots, map, m and tile pair."""
    T = (2 * nbins + 15) // 16
    return -(-npiv // 4096) * maps * (m_max + 1) * (T * T if cross else T * (T + 1) // 2) * 2048


@pytest.fixture
def limit():
    yield lambda size: _lib.load().z3_set_device_alloc_limit(ctypes.c_size_t(size))
    _lib.load().z3_set_device_alloc_limit(ctypes.c_size_t(SIZE_MAX))


def _close(got, ref):
    # FP64 sums of at most 20,000 terms in another order
    assert (got - ref).abs().max() <= 1e-12 * ref.abs().max()


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("npiv,m_max,nbins", [(20000, 8, 10), (4097, 0, 1), (5000, 3, 33)])
def test_contract_under_an_allocation_limit(limit, prec, npiv, m_max, nbins):
    G.say("case: scratch limits, contract", prec, npiv, m_max, nbins)
    g = torch.Generator(device="cuda").manual_seed(npiv)
    A = torch.randn((m_max + 1, 2, nbins, npiv), dtype=torch.float64, device="cuda", generator=g)
    A = A if prec == "fp64" else A.float()
    v = torch.rand(npiv, dtype=torch.float64, device="cuda", generator=g)
    ref = z3.contract(A, v, m_max, nbins, prec)
    limit(_least(npiv, m_max, nbins) - 256)
    with pytest.raises(_lib.Zeta3Error) as err:
        z3.contract(A, v, m_max, nbins, prec)
    assert err.value.status == 2
    limit(_least(npiv, m_max, nbins))
    _close(z3.contract(A, v, m_max, nbins, prec), ref)


def _index(nmaps, nbins):
    xyz = cap_points(5000, 8.0, seed=9).cuda()
    idx = z3.Index(xyz, chord2_edges(theta_edges(arcmin(10.0), arcmin(200.0), nbins, True)))
    x = np.random.default_rng(10).normal(size=(nmaps, 5000))
    idx.set_values(torch.from_numpy(x if nmaps > 1 else x[0]).cuda())
    return idx


@pytest.mark.parametrize("what", ["estimate", "no_self", "maps", "cross"])
def test_capture_in_a_reservation_for_the_least(what):
    G.say("case: scratch limits, capture", what)
    nbins, m_max = 6, 4
    nmaps = 1 if what in ("estimate", "no_self") else 3

    def body(idx, zeta):
        if what in ("estimate", "no_self"):
            z3.estimate_raw(idx, m_max, zeta=zeta, self_pairs=what == "estimate")
        elif what == "maps":
            z3.estimate_maps_raw(idx, m_max, zeta=zeta)
        else:
            z3.estimate_cross_raw(idx, (0, 1, 2), m_max, cyclic=True, zeta=zeta)

    shape = ((3,) if what == "maps" else ()) + (m_max + 1, nbins, nbins, 2)
    ref = torch.zeros(shape, dtype=torch.float64, device="cuda")
    other = _index(nmaps, nbins)
    body(other, ref)
    idx = _index(nmaps, nbins)  # no eager call on this one: only the reservation below
    chunk, sets = 5120, {"maps": 4, "cross": 4}.get(what, 1)
    least = _least(chunk, m_max, nbins, 4 if what == "maps" else 1, what == "cross")
    room = sets * chunk * (m_max + 1) * 2 * nbins * 8 + least
    if what == "no_self":
        room += (chunk // 64 * nbins * 8 + 255) // 256 * 256
    reserved = ctypes.c_size_t()
    _lib.call("z3_index_prepare_capture", idx.handle, room, ctypes.byref(reserved))
    assert reserved.value == room
    zeta = torch.zeros(shape, dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        zeta.zero_()
        body(idx, zeta)
    for _ in range(3):
        graph.replay()
        torch.cuda.synchronize()
        _close(zeta, ref)
    idx.free()
    other.free()
