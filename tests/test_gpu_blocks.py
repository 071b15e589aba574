"""Device memory of an index that is freed while the runtime refuses a device-wide wait (a stream
is being captured): no other index may get it before the work that reads it has ended."""

import ctypes
import time

import numpy as np
import pytest
import torch

import paper_2408_16847_amd as z3
from paper_2408_16847_amd import _lib
from synth import ring_centres
from synth.bins import arcmin, chord2_edges, theta_edges
from tests import gpu_helpers as G

pytestmark = pytest.mark.gpu


def _hip_runtime():
    """The HIP runtime that this process already has loaded."""
    _lib.load()
    hip = ctypes.CDLL(next(ln.split()[-1] for ln in open("/proc/self/maps") if "libamdhip64" in ln))
    hip.hipStreamBeginCapture.argtypes = [ctypes.c_void_p, ctypes.c_int]
    hip.hipStreamEndCapture.argtypes = [ctypes.c_void_p, ctypes.POINTER(ctypes.c_void_p)]
    return hip


def test_index_freed_while_another_stream_captures():
    G.say("case: index freed during a capture")
    hip = _hip_runtime()
    xyz = ring_centres(96).cuda()
    n = xyz.shape[1]
    E = chord2_edges(theta_edges(arcmin(60.0), arcmin(600.0), 8, True))
    rng = np.random.default_rng(7)
    x, y = (torch.from_numpy(rng.normal(size=n)).cuda() for _ in range(2))
    mirrored = xyz.flip(0).contiguous()
    M = 10
    expect = []
    for pos, val in ((xyz, x), (mirrored, y)):
        idx = z3.Index(pos, E)
        idx.set_values(val)
        expect.append(z3.estimate_raw(idx, M).cpu())
        idx.free()
    torch.cuda.synchronize()

    busy, capturing, other = torch.cuda.Stream(), torch.cuda.Stream(), torch.cuda.Stream()
    first = z3.Index(xyz, E)
    first.set_values(x)
    zeta = torch.zeros((M + 1, 8, 8, 2), dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    with torch.cuda.stream(busy):
        for _ in range(8):  # tens of milliseconds of work that reads the first index
            zeta.zero_()
            z3.estimate_raw(first, M, zeta=zeta)
    # mode 0 (global): the runtime refuses calls that wait for the device
    assert hip.hipStreamBeginCapture(capturing.cuda_stream, 0) == 0
    _lib.load().z3_index_free(first._h)
    first._h = ctypes.c_void_p()
    G.say("  the wait's status:", _lib.load().z3_last_error().decode())
    graph = ctypes.c_void_p()
    hip.hipStreamEndCapture(capturing.cuda_stream, ctypes.byref(graph))
    hip.hipGetLastError()
    with torch.cuda.stream(other):
        second = z3.Index(mirrored, E)
        second.set_values(y)
        got = z3.estimate_raw(second, M)
    torch.cuda.synchronize()
    assert torch.equal(zeta.cpu(), expect[0])
    assert torch.equal(got.cpu(), expect[1])
    second.free()
    # the device is idle: the first index's memory is free for the next one
    third = z3.Index(xyz, E)
    third.set_values(x)
    assert torch.equal(z3.estimate_raw(third, M).cpu(), expect[0])
    third.free()


def test_memory_of_freed_indexes_can_be_given_back():
    G.say("case: index memory given back")
    xyz = ring_centres(256).cuda()
    n = xyz.shape[1]
    x = torch.zeros(n, dtype=torch.float64, device="cuda")
    z3.release_index_memory()
    torch.cuda.synchronize()
    time.sleep(0.5)  # the driver's figure follows a free with some delay
    before = torch.cuda.mem_get_info()[0]
    idx = z3.Index(xyz, chord2_edges(theta_edges(arcmin(60.0), arcmin(600.0), 8, True)))
    idx.set_values(x)
    idx.free()
    held = before - torch.cuda.mem_get_info()[0]
    G.say("  held after the index was freed:", held)
    assert held > 100 * n  # 64 B of records a point alone, and the build's arrays
    z3.release_index_memory()
    for _ in range(40):
        held = before - torch.cuda.mem_get_info()[0]
        if held < 8 << 20:
            break
        time.sleep(0.05)
    assert held < 8 << 20  # the runtime's own rounding at most
