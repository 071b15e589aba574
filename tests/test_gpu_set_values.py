"""z3_index_set_values waits for earlier work on its stream, also where it attaches the first
values, and is refused on a stream that is being captured."""

import ctypes

import pytest
import torch

import paper_2408_16847_amd as z3
from paper_2408_16847_amd import _lib
from synth import cap_points
from synth.bins import arcmin, chord2_edges, theta_edges
from tests import gpu_helpers as G

pytestmark = pytest.mark.gpu

E = chord2_edges(theta_edges(arcmin(10.0), arcmin(200.0), 4, True))


@pytest.mark.parametrize("attached", [False, True])
def test_waits_for_earlier_work_on_the_stream(attached):
    G.say("case: set_values waits", attached)
    x = torch.ones(1000, dtype=torch.float64, device="cuda")
    idx = z3.Index(cap_points(1000, 5.0, seed=1).cuda(), E)
    if attached:
        idx.set_values(x)
    a = torch.randn(8192, 8192, device="cuda")
    b = torch.empty_like(a)
    torch.mm(a, a, out=b)
    torch.cuda.synchronize()
    stream, done = torch.cuda.Stream(), torch.cuda.Event()
    with torch.cuda.stream(stream):
        for _ in range(30):  # a quarter of a second
            torch.mm(a, a, out=b)
        done.record()
        idx.set_values(x)
        assert done.query()
    torch.cuda.synchronize()
    idx.free()


@pytest.mark.parametrize("attached", [False, True])
def test_refused_on_a_capturing_stream(attached):
    G.say("case: set_values on a capturing stream", attached)
    lib = _lib.load()
    hip = ctypes.CDLL(next(ln.split()[-1] for ln in open("/proc/self/maps") if "libamdhip64" in ln))
    hip.hipStreamBeginCapture.argtypes = [ctypes.c_void_p, ctypes.c_int]
    hip.hipStreamEndCapture.argtypes = [ctypes.c_void_p, ctypes.POINTER(ctypes.c_void_p)]
    xyz = cap_points(1000, 5.0, seed=1).cuda()
    x = torch.ones(1000, dtype=torch.float64, device="cuda")
    z3.Index(xyz, E).set_values(x).free()  # memory for the arrays is at hand
    idx = z3.Index(xyz, E)
    if attached:
        idx.set_values(x)
        before = z3.estimate(idx, 3)
    torch.cuda.synchronize()
    stream, graph = torch.cuda.Stream(), ctypes.c_void_p()
    assert hip.hipStreamBeginCapture(stream.cuda_stream, 0) == 0
    st = lib.z3_index_set_values(idx.handle, 1, ctypes.c_void_p(x.data_ptr()), ctypes.c_void_p(stream.cuda_stream))
    hip.hipStreamEndCapture(stream.cuda_stream, ctypes.byref(graph))
    hip.hipGetLastError()
    assert st == 3, lib.z3_last_error()
    if attached:
        after = z3.estimate(idx, 3)
        assert after[1] == before[1] and (after[0] == before[0]).all()
    idx.free()
