"""Registers of the step kernels as built, from the code objects in the
library: the BF16 kernels without position noise over contiguous groups keep
six waves per SIMD (at most 80 of its 512 VGPRs each) and no scratch; the view
step over windows of 128 and 256 keeps five (96)."""
import os
import re
import struct
import subprocess

import pytest

import paper_2601_16736_amd as gs

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(data):
    at = data.find(MAGIC)
    while at >= 0:
        entries, = struct.unpack_from("<Q", data, at + 24)
        o = at + 32
        for _ in range(entries):
            off, size, length = struct.unpack_from("<QQQ", data, o)
            name = data[o + 24:o + 24 + length]
            o += 24 + length
            if b"gfx950" in name:
                yield data[at + off:at + off + size]
        at = data.find(MAGIC, at + 1)


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """(VGPRs, scratch bytes) of each kernel by its mangled name."""
    if not os.path.exists(READELF):
        pytest.skip("no llvm-readelf")
    lib = os.path.join(os.path.dirname(gs.__file__), "libgsopt.so")
    found = {}
    with open(lib, "rb") as f:
        objects = list(_code_objects(f.read()))
    for k, obj in enumerate(objects):
        path = tmp_path_factory.mktemp("co") / f"{k}.elf"
        path.write_bytes(obj)
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
        for block in re.split(r"\n\s*- \.ag?pr_count|\n\s*- \.args", notes)[1:]:
            field = {m[1]: m[2] for m in re.finditer(r"\.(name|vgpr_count|private_segment_fixed_size):\s+(\S+)", block)
                     if m[1] != "name" or m[2].startswith("_ZN2gs")}
            if "name" in field:
                found[field["name"]] = (int(field["vgpr_count"]), int(field["private_segment_fixed_size"]))
    return found


@pytest.mark.parametrize("pattern,most,frame", [
    (r"16step_view_kernelILb1ELi(32|64)ELb0ELb[01]ELb0ENS_[78]KCameras?E", 80, 0),
    (r"16step_view_kernelILb1ELi(128|256)ELb0ELb[01]ELb0ENS_[78]KCameras?E", 96, 36),
    (r"11step_kernelILb1ELi[123]ELi(32|64|128|256|512)ELb0ELb0EE", 80, 0)])
def test_bf16_step_kernels_keep_their_waves(kernels, pattern, most, frame):
    picked = {k: v for k, v in kernels.items() if re.search(pattern, k)}
    assert len(picked) >= 8
    for name, (vgprs, scratch) in picked.items():
        assert vgprs <= most and scratch <= frame, (name, vgprs, scratch)
