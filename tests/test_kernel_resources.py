"""Registers and LDS of the passes over K, from the built library's own kernel descriptions: two workgroups of four waves have to fit
a CU (512 registers per lane and SIMD, 160 KB of LDS), else nobody covers a workgroup's LDS and MFMA phases; with 64 dims and
chunks of 1024 tokens three."""
import os
import re
import struct
import subprocess

import pytest

from paper_2503_08879_amd.build import LIB

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
FILTER, PARTIALS = 1, 2  # ScoreMode


def device_objects(data):
    """The gfx950 code objects of a library: every source file's offload bundle holds one."""
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = data.find(magic)
    while at >= 0:
        n, pos = struct.unpack_from("<Q", data, at + 24)[0], at + 32
        for _ in range(n):
            offset, size, length = struct.unpack_from("<QQQ", data, pos)
            if b"gfx950" in data[pos + 24:pos + 24 + length]:
                yield data[at + offset:at + offset + size]
            pos += 24 + length
        at = data.find(magic, at + 32)


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    if not os.path.exists(READELF):
        pytest.skip("no llvm-readelf")
    out = {}
    with open(LIB, "rb") as f:
        data = f.read()
    for i, obj in enumerate(device_objects(data)):
        path = tmp_path_factory.mktemp("co") / f"{i}.co"
        path.write_bytes(obj)
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
        for part in re.split(r"\n  - \.a", notes)[1:]:
            field = dict(re.findall(r"\.(\w+): +(\S+)", ".a" + part))
            out[field["symbol"].strip("'")] = field
    return out


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("heads", [4, 8, 16])
@pytest.mark.parametrize("mode", [FILTER, PARTIALS])
def test_workgroups_per_cu(kernels, d, heads, mode):
    mine = {name: f for name, f in kernels.items() if f"score_mfma_kernelILi{d}ELi{heads}ELi{mode}E" in name}
    assert len(mine) == 6  # pages or not, chunks of 256, 512 and 1024 tokens
    for name, f in mine.items():
        fit = 3 if d == 64 and re.search(r"Lb[01]ELi4EE", name) else 2
        assert int(f["vgpr_count"]) <= 512 // fit // 8 * 8, f  # both kinds of vector registers, in units of 8
        assert int(f["group_segment_fixed_size"]) <= 160 * 1024 // fit, f
        if fit == 2:
            assert int(f["vgpr_spill_count"]) == 0, f
