"""The index build at the edges of its kernels, against the grid's definition in NumPy: the index
order (band, then cell, then catalogue order), its number of bands and cells, and the pairs it
finds; indexes made, freed and made again, whose memory the library keeps between them."""

import math
import threading

import numpy as np
import pytest
import torch

import paper_2408_16847_amd as z3
from synth import cap_points, plane_points, ring_centres
from synth.bins import chord2_edges, theta_edges
from tests import gpu_helpers as G

pytestmark = pytest.mark.gpu

E = chord2_edges(theta_edges(math.radians(0.5), math.radians(4.0), 3, True))


def _order(band, phi, ncell_per_point=4):
    """Index order of points in `band` with longitude `phi`: cells of equal longitude, four per
    point of the band, points of a cell in catalogue order."""
    count = np.bincount(band, minlength=band.max() + 1)
    ncell = np.maximum(1, ncell_per_point * count)[band]
    cell = np.clip(np.floor(phi * (ncell / (2.0 * math.pi))).astype(np.int64), 0, ncell - 1)
    return np.lexsort((np.arange(len(band)), cell, band))


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 1023, 1025, 5000])
@pytest.mark.parametrize("cell", [0.05, 0.002, 0.0005])  # up to, and beyond, the bands held in LDS
def test_random_order_catalogue(n, cell):
    G.say("case: index build", n, cell)
    xyz = cap_points(n, 12.0, seed=n).numpy()
    idx = G.build(xyz, np.ones(n), E, cell_size=cell)
    th = np.arctan2(np.sqrt(xyz[0] ** 2 + xyz[1] ** 2), xyz[2])
    phi = np.arctan2(xyz[1], xyz[0])
    phi = np.where(phi < 0, phi + 2 * math.pi, phi)
    nbands = math.ceil(math.pi / cell)
    band = np.minimum((th * (1.0 / cell)).astype(np.int64), nbands - 1)
    info = idx.info()
    assert info["nbands"] == nbands
    assert info["ncells"] == np.maximum(1, 4 * np.bincount(band, minlength=nbands)).sum()
    assert np.array_equal(G.perm(idx), _order(band, phi))


def test_map_order_many_bands():
    G.say("case: index build, map order")
    ring = ring_centres(40)
    xyz = ring.numpy()
    for cell in (0.0, 0.004, 0.0011):
        idx = G.build(xyz, np.ones(xyz.shape[1]), E, cell_size=cell)
        p = G.perm(idx)
        assert np.array_equal(np.sort(p), np.arange(xyz.shape[1]))
        a, W, N, H = G.gpu_multipoles(idx, 2, 0, 400, norm="none")
        ao, Wo, No, _, Ho = G.oracle_multipoles(xyz, np.ones(xyz.shape[1]), np.ones(xyz.shape[1]), E, 2, p[:400])
        assert np.array_equal(N, No) and np.array_equal(H, Ho)


def test_plane_strips():
    G.say("case: index build, plane")
    xy = plane_points(50, seed=3).numpy()
    idx = z3.Index(torch.from_numpy(xy).cuda(), np.linspace(1.0, 3.0, 4) ** 2, cell_size=1.7, planar=True)
    y = xy[1] - xy[1].min()
    band = np.minimum((y * (1.0 / 1.7)).astype(np.int64), int(y.max() / 1.7))
    perm = idx.perm().cpu().numpy()
    assert np.array_equal(band[perm], np.sort(band))
    assert idx.info()["nbands"] == int(y.max() / 1.7) + 1


def test_made_and_freed_on_streams_and_threads():
    # every index takes its memory from blocks that earlier ones gave back; none may see another's
    G.say("case: index build, reuse")
    sizes = (3000, 700, 1500, 2999)
    ref = {}
    for n in sizes:
        xyz = cap_points(n, 9.0, seed=n)
        x = np.random.default_rng(n).normal(size=n)
        idx = G.build(xyz.numpy(), x, E)
        ref[n] = (xyz.cuda(), torch.from_numpy(x).cuda(), z3.estimate(idx, 5))
        idx.free()
    torch.cuda.synchronize()
    bad = []

    def work(k):
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            for r in range(6):
                n = sizes[(k + r) % len(sizes)]
                xyz, x, (z, p) = ref[n]
                idx = z3.Index(xyz, E)
                idx.set_values(x)
                idx.set_values(x)  # replaces the values attached before
                got, pairs = z3.estimate(idx, 5)
                if pairs != p or not np.array_equal(got, z):
                    bad.append((k, r, n))
                idx.free()

    threads = [threading.Thread(target=work, args=(k,)) for k in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad


@pytest.mark.parametrize("turn", [False, True])
def test_crowded_cells(turn):
    # stacks of 300 points at 50 positions, one stack after the other or one point of each in turn
    G.say("case: index build, stacks", turn)
    base = cap_points(50, 9.0, seed=6).numpy()
    xyz = np.ascontiguousarray(np.tile(base, (1, 300)) if turn else np.repeat(base, 300, axis=1))
    idx = G.build(xyz, np.ones(xyz.shape[1]), E, cell_size=0.05)
    th = np.arctan2(np.sqrt(xyz[0] ** 2 + xyz[1] ** 2), xyz[2])
    phi = np.arctan2(xyz[1], xyz[0])
    band = np.minimum((th * (1.0 / 0.05)).astype(np.int64), math.ceil(math.pi / 0.05) - 1)
    assert np.array_equal(G.perm(idx), _order(band, np.where(phi < 0, phi + 2 * math.pi, phi)))
    idx.free()
