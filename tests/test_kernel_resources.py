"""What the compiler has given the kernels of the built library, read from the metadata of its code objects: registers decide how
many workgroups a compute unit holds, and a spill is a trip to memory."""
import os
import re
import shutil
import struct
import subprocess

import pytest

import paper_2008_12260_amd as px

READELF = shutil.which("llvm-readelf") or "/opt/rocm/llvm/bin/llvm-readelf"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{mangled name: {field: value}} of every kernel in the library."""
    if not os.path.exists(px.LIB_PATH):
        pytest.skip("the library has not been built")
    data, found, at = open(px.LIB_PATH, "rb").read(), {}, 0
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    while (at := data.find(magic, at)) >= 0:
        entry = at + len(magic) + 8
        for _ in range(struct.unpack_from("<Q", data, at + len(magic))[0]):
            offset, size, length = struct.unpack_from("<QQQ", data, entry)
            target = data[entry + 24:entry + 24 + length].decode()
            entry += 24 + length
            if size == 0 or "gfx950" not in target:
                continue
            path = tmp_path_factory.mktemp("code") / "object"
            path.write_bytes(data[at + offset:at + offset + size])
            notes = subprocess.run([READELF, "--notes", str(path)], check=True, capture_output=True, text=True).stdout
            for block in notes.split("  - .agpr_count:")[1:]:
                name = re.search(r"^ +\.name: +(\S+)$", block, re.M).group(1)
                found[name] = {k: int(v) for k, v in re.findall(r"^ +\.(\w+): +(\d+)$", block, re.M)}
        at += len(magic)
    assert len(found) > 50
    return found


@pytest.mark.parametrize("which,instances,spilled", [
    ("pairs_kernelILi0ELb0ELb0E", 3, 16),           # the sampling argmax of every pair
    ("pairs_kernelILi0ELb0ELb1E", 3, 32),           # rows looked up, the sampling argmax for those beyond the tables
    ("pairs_kernelILi16ELb0ELb1E", 3, 48)])         # the same, the grid's
def test_rows_priced_in_place_spill_little(kernels, which, instances, spilled):
    """Bytes a lane: more and a pass over a few thousand pairs is up to a tenth slower, whether or not it meets such a row."""
    names = [n for n in kernels if which in n]
    assert len(names) == instances
    for n in names:
        assert kernels[n]["private_segment_fixed_size"] <= spilled, n


def test_a_compute_unit_holds_three_children(kernels):
    names = [n for n in kernels if "child_kernel" in n]
    assert len(names) == 6
    for n in names:
        # eight wavefronts a workgroup, two on each of four SIMDs of 512 registers, given out in eights
        assert 512 // (-(-kernels[n]["vgpr_count"] // 8) * 8) >= 6, n
