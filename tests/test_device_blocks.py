"""The device blocks that the library keeps between indexes, on the CPU: csrc/z3_blocks.hip
compiled for the host against a stand-in of the runtime calls it makes
(tests/sanitize/blocks_checks.cpp), under the address and undefined-behaviour sanitizers and
under the thread sanitizer."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
OUT = os.path.join(ROOT, "_build", "sanitize")
CLANG = "/opt/rocm/llvm/bin/clang++"


@pytest.mark.parametrize("sanitizer", ["address,undefined", "thread"])
def test_block_reaches_a_new_owner_only_after_a_wait(sanitizer):
    if not (os.path.exists(CLANG) or shutil.which(CLANG)):
        pytest.skip("ROCm clang not available")
    os.makedirs(OUT, exist_ok=True)
    exe = os.path.join(OUT, "blocks_" + sanitizer.split(",")[0])
    src = os.path.join(ROOT, "paper_2408_16847_amd", "csrc")
    cmd = [CLANG, "-x", "c++", "-std=c++17", "-O1", "-g", "-D__HIP_PLATFORM_AMD__", "-Wno-unused-result",
           f"-fsanitize={sanitizer}", "-I", "/opt/rocm/include", "-I", os.path.join(ROOT, "include"),
           "-I", src, os.path.join(src, "z3_blocks.hip"), os.path.join(ROOT, "tests", "sanitize", "blocks_checks.cpp"),
           "-lpthread", "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "block checks ok" in r.stdout, r.stdout + r.stderr
