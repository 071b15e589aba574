"""The FFTLog pass length on the CPU (tests/sanitize/fftlog_pass_checks.cpp), and the sizes that the
entry point refuses before any device work."""

import ctypes
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
OUT = os.path.join(ROOT, "_build", "sanitize")


def test_pass_length_keeps_offsets_in_range():
    if not shutil.which("g++"):
        pytest.skip("g++ not available")
    os.makedirs(OUT, exist_ok=True)
    exe = os.path.join(OUT, "fftlog_pass")
    cmd = ["g++", "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all",
           "-I", os.path.join(ROOT, "paper_2408_16847_amd", "csrc"),
           os.path.join(ROOT, "tests", "sanitize", "fftlog_pass_checks.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and "pass checks ok" in r.stdout, r.stdout + r.stderr


@pytest.mark.parametrize("nchi,status", [(522248, 5), (2 ** 31 - 1, 5), (522247, 2)])
def test_sizes_refused_before_device_work(nchi, status):
    from paper_2408_16847_amd import _lib
    lib = _lib.load()
    fake, nu = ctypes.c_void_p(0x1000), (ctypes.c_double * 4)(-1.3, -2.5, -1.3, -1.3)
    try:
        lib.z3_set_device_alloc_limit(0)  # a size that is taken ends at the workspace's allocation
        st = lib.z3_fftlog_a_functions(4096, fake, 1e-6, 30.0, nu, nchi, 1e-4, 60.0, 1, fake, 1, fake, fake, None,
                                       ctypes.c_size_t(0), None)
    finally:
        lib.z3_set_device_alloc_limit(ctypes.c_size_t(-1).value)
    assert st == status, lib.z3_last_error()
