"""Registers of the hop kernel as it was built: what decides how many wavefronts stay on a SIMD (512 registers, taken
in eights)."""
import os
import re
import struct
import subprocess

import pytest

import paper_2207_12000_amd as gp

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects():
    """The gfx950 code objects inside the library: every bundle is the magic, a count, and (offset, size, name) entries."""
    data = open(gp.LIB_PATH, "rb").read()
    for m in re.finditer(MAGIC, data):
        p = m.start() + len(MAGIC)
        count, p = struct.unpack_from("<Q", data, p)[0], p + 8
        for _ in range(count if count < 8 else 0):
            offset, size, length = struct.unpack_from("<QQQ", data, p)
            name, p = data[p + 24:p + 24 + length], p + 24 + length
            if name.endswith(b"gfx950"):
                yield data[m.start() + offset:m.start() + offset + size]


@pytest.mark.skipif(not os.path.exists(READELF), reason="llvm-readelf not found")
def test_weighted_hops_over_two_columns_keep_five_wavefronts(tmp_path):
    registers = {}
    for i, code in enumerate(code_objects()):
        path = tmp_path / f"{i}.co"
        path.write_bytes(code)
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
        for entry in re.split(r"\n  - \.agpr_count", notes)[1:]:
            name = re.search(r"\.name:\s+(\S+)", entry).group(1)
            m = re.search(r"gp_hop_segmentsI([ft])Li(\d)ELi(\d+)ELi(\d)ELi(\d)E", name)
            if m:
                registers[m.groups()] = int(re.search(r"\.vgpr_count:\s+(\d+)", entry).group(1))
    assert 512 // 8 // ((registers["f", "2", "8", "1", "2"] + 7) // 8) >= 5


@pytest.fixture(scope="module")
def wavefronts(tmp_path_factory):
    """Wavefronts per SIMD (eight at most) of every instance of the hop and the fix-up kernel that copies no rows, by its
    template arguments."""
    if not os.path.exists(READELF):
        pytest.skip("llvm-readelf not found")
    found = {}
    for i, code in enumerate(code_objects()):
        path = tmp_path_factory.mktemp("co") / f"{i}.co"
        path.write_bytes(code)
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
        for entry in re.split(r"\n  - \.agpr_count", notes)[1:]:
            name = re.search(r"\.name:\s+(\S+)", entry).group(1)
            m = re.search(r"gp_(hop_segments|fixup_rows)I([ft])Li(\d)ELi(\d+)ELi(\d)E(?:Li(\d)E)?", name)
            if m:
                assert int(re.search(r"\.vgpr_spill_count:\s+(\d+)", entry).group(1)) == 0, name
                found[m.groups()] = min(8, 512 // 8 // ((int(re.search(r"\.vgpr_count:\s+(\d+)", entry).group(1)) + 7) // 8))
    return found


def test_fix_ups_keep_six_wavefronts(wavefronts):
    assert all(count >= 6 for name, count in wavefronts.items() if name[0] == "fixup_rows")


def test_launches_that_copy_no_rows_lose_no_wavefront_to_those_that_do(wavefronts):
    assert wavefronts["hop_segments", "t", "2", "16", "1", "0"] >= 7  # 72 registers; 73 with the branches for copies
