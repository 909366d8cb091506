"""What the kernels of the built library take, from the notes of its own code
objects: a kernel past its line runs, but with fewer waves or with registers in
memory."""
import os
import re
import struct
import subprocess

import pytest

from paper_2003_13493_amd import fastgrid

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
FIELDS = ("private_segment_fixed_size", "sgpr_spill_count", "vgpr_count", "vgpr_spill_count")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """Mangled kernel name -> fields, over the library's gfx950 code objects."""
    with open(fastgrid.LIB_PATH, "rb") as f:
        data = f.read()
    out, at = {}, data.find(b"\x7fELF", 4)
    path = str(tmp_path_factory.mktemp("code") / "object")
    while at >= 0:
        if struct.unpack_from("<H", data, at + 18)[0] == 224:   # EM_AMDGPU
            size = struct.unpack_from("<Q", data, at + 40)[0] + \
                struct.unpack_from("<H", data, at + 58)[0] * struct.unpack_from("<H", data, at + 60)[0]
            with open(path, "wb") as f:
                f.write(data[at:at + size])
            notes = subprocess.run([READELF, "--notes", path], capture_output=True, text=True, check=True).stdout
            for entry in re.split(r"\n  - \.agpr_count", notes)[1:]:
                name = re.search(r"\n    \.name: +(\S+)", entry).group(1)
                out[name] = {k: int(re.search(rf"\n    \.{k}: +(\d+)", entry).group(1)) for k in FIELDS}
        at = data.find(b"\x7fELF", at + 4)
    assert out
    return out


def one(kernels, name):
    found = [k for k in kernels if name in k]
    assert len(found) == 1, (name, found)
    return kernels[found[0]]


def test_batches_without_whole_regions(kernels):
    """Their kernel keeps general geometry and group entries without spilling much of either."""
    k = one(kernels, "detect_batch_any_kernel")
    assert k["vgpr_spill_count"] == 0 and k["private_segment_fixed_size"] == 0
    assert k["sgpr_spill_count"] <= 30


def test_wide_workgroups(kernels):
    """Two workgroups of 512 threads on a CU take 128 registers of a thread at most."""
    for name in ("detect_batch_any_kernel", "detect_batch_generic_kernelILb1E"):
        assert one(kernels, name)["vgpr_count"] <= 128


def test_generic_batches(kernels):
    """The general geometry of regions of any size stays clear of the scalar registers."""
    k = one(kernels, "detect_batch_generic_kernelILb0E")
    assert k["vgpr_spill_count"] == 0 and k["private_segment_fixed_size"] == 0
    assert k["sgpr_spill_count"] <= 80


def test_nothing_in_scratch_memory(kernels):
    """No kernel keeps a value in private memory, by a spill or by an address taken."""
    assert {k: v for k, v in kernels.items() if v["private_segment_fixed_size"] or v["vgpr_spill_count"]} == {}
