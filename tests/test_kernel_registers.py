"""Registers of the many-map kernel, from the metadata of the library's own code objects: in the forms
that request the next candidate's values ahead, spilled registers are reloaded for every candidate
and cost more than the request gains.  (CPU only: nothing is launched.)"""

import os
import re
import struct
import subprocess

import pytest

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(data):
    """The gfx950 code objects of every offload bundle in `data`."""
    at = data.find(MAGIC)
    while at >= 0:
        (count,) = struct.unpack_from("<Q", data, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", data, p)
            target = data[p + 24:p + 24 + length]
            p += 24 + length
            if b"gfx950" in target and size:
                yield data[at + offset:at + offset + size]
        at = data.find(MAGIC, at + 1)


def _spills(tmp_path, kernel):
    """{mangled name: spilled vector registers} of the kernels whose name holds `kernel`."""
    from paper_2408_16847_amd import _lib
    out = {}
    for k, blob in enumerate(_code_objects(open(_lib.LIB_PATH, "rb").read())):
        if kernel.encode() not in blob:
            continue
        path = tmp_path / f"{k}.co"
        path.write_bytes(blob)
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True).stdout
        for entry in re.split(r"\n\s+- \.", notes):
            name = re.search(r"\.name:\s+(\S+)", entry)
            spill = re.search(r"\.vgpr_spill_count:\s+(\d+)", entry)
            if name and spill and kernel in name.group(1):
                out[name.group(1)] = int(spill.group(1))
    return out


def test_many_map_forms_do_not_spill_in_the_candidate_loop(tmp_path):
    if not os.path.exists(READELF):
        pytest.skip("llvm-readelf not available")
    spills = _spills(tmp_path, "k_multipoles_maps")
    form = re.compile(r"k_multipoles_mapsILi(\d+)ELb([01])ELi(\d)ELb([01])E")
    seen = set()
    for name, spill in spills.items():
        M, f32, K, lists = (int(v) for v in form.search(name).groups())
        seen.add((M, f32, K, lists))
        if K == 2 or (K == 4 and M in (5, 6, 7, 8)):
            assert spill == 0, (M, f32, K, lists, spill)
    assert len(seen) == 2 * 2 * (17 + 12 + 5)
