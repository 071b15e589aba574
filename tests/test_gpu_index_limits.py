"""Catalogues at the limits of the index build: refused before any array over the cells exists, and
built with cell arrays of exactly the cells there are where an allocation limit leaves no more."""

import ctypes
import math

import numpy as np
import pytest
import torch

import paper_2408_16847_amd as z3
from paper_2408_16847_amd import _lib
from synth import cap_points
from synth.bins import arcmin, chord2_edges, theta_edges
from tests import gpu_helpers as G

pytestmark = pytest.mark.gpu

E = chord2_edges(theta_edges(arcmin(10.0), arcmin(200.0), 4, True))
SIZE_MAX = ctypes.c_size_t(-1).value


@pytest.fixture
def limit():
    yield lambda size: _lib.load().z3_set_device_alloc_limit(ctypes.c_size_t(size))
    _lib.load().z3_set_device_alloc_limit(ctypes.c_size_t(SIZE_MAX))


def test_band_of_too_many_points_is_refused_before_its_cells(limit):
    # 2^26 points spread over one band's longitudes; their cells alone would be 1 GiB
    G.say("case: index limits, full band")
    n = 1 << 26
    phi = torch.arange(n, dtype=torch.float64, device="cuda") * (2.0 * math.pi / n)
    xyz = torch.stack([torch.cos(phi), torch.sin(phi), torch.zeros_like(phi)])
    limit(9 * n)  # the arrays over points fit, 8 bytes a point
    with pytest.raises(z3._lib.Zeta3Error) as err:
        z3.Index(xyz, E, cell_size=4.0)
    assert err.value.status == 4 and str(n) in str(err.value)


def test_exact_cell_arrays_under_an_allocation_limit(limit):
    G.say("case: index limits, exact cells")
    n = 1000
    pos = cap_points(n, 10.0, seed=5).cuda()
    x = torch.from_numpy(np.random.default_rng(4).normal(size=n)).cuda()
    idx = z3.Index(pos, E, cell_size=0.02)
    cells = idx.info()["ncells"]
    assert cells < 4 * n + idx.info()["nbands"]
    idx.set_values(x)
    ref, perm = z3.estimate(idx, 4), idx.perm()
    idx.free()
    limit(4 * cells)  # one entry too few
    with pytest.raises(z3._lib.Zeta3Error) as err:
        z3.Index(pos, E, cell_size=0.02)
    assert err.value.status == 2
    limit(4 * (cells + 1))
    idx = z3.Index(pos, E, cell_size=0.02)
    limit(SIZE_MAX)
    assert idx.info()["ncells"] == cells and torch.equal(idx.perm(), perm)
    idx.set_values(x)
    got = z3.estimate(idx, 4)
    assert got[1] == ref[1] and np.array_equal(got[0], ref[0])
    idx.free()
