"""Registers of the built kernels, from the metadata of the code objects in libtaq.so. No GPU."""
import glob
import os
import re
import shutil
import subprocess

import pytest

from paper_2603_22943_amd import build as B

TOOLS = os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(B.hipcc_path()))), "llvm", "bin")


@pytest.fixture(scope="module")
def metadata(tmp_path_factory):
    """{kernel: {field: value}}"""
    folder = str(tmp_path_factory.mktemp("objects"))
    lib = shutil.copy(B.LIB, folder)  # (the code objects are written beside it)
    subprocess.run([os.path.join(TOOLS, "llvm-objdump"), "--offloading", lib], check=True, capture_output=True)
    kernels = {}
    for part in glob.glob(lib + ".*amdgcn*"):
        notes = subprocess.run([os.path.join(TOOLS, "llvm-readelf"), "--notes", part], check=True, capture_output=True, text=True).stdout
        for entry in notes.split("  - .agpr_count:")[1:]:
            fields = dict(re.findall(r"^    \.(\w+): +(\S+)$", entry, re.M))
            kernels[fields["name"]] = fields
    assert len(kernels) > 300
    return kernels


@pytest.mark.parametrize("kernel", ["rowquant_op_kernel", "rowquant_f16_kernel", "kv_prep_kernel"])
def test_row_quantizers_leave_room_for_eight_wavefronts(metadata, kernel):
    """512 registers of a SIMD's lane: 8192 rows are 8 wavefronts a SIMD, and with 73 registers ran as two rounds of six."""
    found = [int(f["vgpr_count"]) for name, f in metadata.items() if kernel in name]
    assert found and max(found) <= 64, found


def test_scratch(metadata):
    """Bytes of scratch a lane: none but where it is known, and known to cost nothing (csrc/taq_fused_kernel.h, FusedCfg and SELECT)."""
    spilled = {name: int(f["private_segment_fixed_size"]) for name, f in metadata.items() if int(f["private_segment_fixed_size"])}
    known = {}
    for grid in range(3):
        for d, heads, tiles, rows, most in ((64, 10, 3, 0, 60), (64, 10, 3, 1, 52), (80, 8, 4, 1, 20)):
            known[f"fused_block_kernelILi{d}ELi{heads}ELi{tiles}ELi{grid}ELi{16 * tiles}ELi5ELb0ELb{rows}EE"] = most
    for name, size in spilled.items():
        assert any(k in name and size <= most for k, most in known.items()), (name, size)
