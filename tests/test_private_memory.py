"""Registers of the built kernels: what their metadata in libaquakv.so says about vector registers kept in private memory."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2501_19392_amd import binding as B

LLVM = "/opt/rocm/llvm/bin/"
# kernel: bytes of private memory a thread may have
ALLOWED = {"exact_gram_kernel": 228, "weighted_values_kernelIfLi4ELi4E": 16, "fused_wide_encode_kernelILi16E": 16, "fused_wide_encode_kernelILi256E": 16}


def test_kernels_keep_their_registers(tmp_path):
    if not os.path.exists(LLVM + "llvm-readelf"):
        pytest.skip("no llvm-readelf")
    shutil.copy(B.LIB_PATH, tmp_path / "lib.so")
    subprocess.run([LLVM + "llvm-objdump", "--offloading", "lib.so"], cwd=tmp_path, check=True, capture_output=True)
    kernels = 0
    for obj in tmp_path.glob("lib.so.*gfx950"):
        notes = subprocess.run([LLVM + "llvm-readelf", "--notes", str(obj)], check=True, capture_output=True, text=True).stdout
        for kernel in re.split(r"^  - \.agpr_count", notes, flags=re.M)[1:]:
            field = lambda name: re.search(rf"\.{name}:\s+(\S+)", kernel)[1]
            kernels += 1
            most = next((size for name, size in ALLOWED.items() if name in field("name")), 0)
            assert int(field("private_segment_fixed_size")) <= most, (field("name"), field("private_segment_fixed_size"), field("vgpr_spill_count"))
    assert kernels > 400
