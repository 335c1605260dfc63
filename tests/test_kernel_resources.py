"""Registers and scratch memory of the kernel that touches every coordinate, from the built library's own metadata."""
import os
import re
import struct
import subprocess

import pytest

from paper_2011_06495_amd import binding as B
from paper_2011_06495_amd import build as mv_build

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(blob):
    """The gfx950 objects of every offload bundle in a library."""
    at = blob.find(BUNDLE)
    while at >= 0:
        (n,) = struct.unpack_from("<Q", blob, at + len(BUNDLE))
        p = at + len(BUNDLE) + 8
        for _ in range(n):
            offset, size, length = struct.unpack_from("<QQQ", blob, p)
            target = blob[p + 24:p + 24 + length]
            p += 24 + length
            if target.endswith(b"gfx950") and size:
                yield blob[at + offset:at + offset + size]
        at = blob.find(BUNDLE, at + 1)


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    if not os.path.exists(READELF):
        pytest.skip("no llvm-readelf")
    if not os.path.exists(B.LIB_PATH):
        mv_build.build_lib()
    found = {}
    for i, obj in enumerate(code_objects(open(B.LIB_PATH, "rb").read())):
        path = tmp_path_factory.mktemp("objects") / ("%d.elf" % i)
        path.write_bytes(obj)
        notes = subprocess.run([READELF, "--notes", str(path)], check=True, capture_output=True, text=True).stdout
        for part in re.split(r"\n  - \.(?=agpr_count|args)", notes)[1:]:
            figures = {k: int(v) for k, v in re.findall(r"\.(\w+):\s+(\d+)\s*$", part, re.M)}
            found[re.search(r"\.symbol:\s+(\S+?)\.kd", part).group(1)] = figures
    return found


def test_streaming_pass_keeps_eight_waves_to_a_simd(kernels):
    """512 registers a lane and SIMD, so 64 for each of eight waves; 160 KB of LDS for the four workgroups of a unit."""
    streams = {name: k for name, k in kernels.items() if "mv_stream_collect" in name}
    assert len(streams) == 2, sorted(kernels)
    for name, k in streams.items():
        assert k["vgpr_count"] <= 64, "%s: %d registers" % (name, k["vgpr_count"])
        assert k["vgpr_spill_count"] == 0 and k["private_segment_fixed_size"] == 0, name
        assert 4 * k["group_segment_fixed_size"] <= 160 * 1024, name
