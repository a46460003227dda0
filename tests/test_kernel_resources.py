"""Registers of the built kernels: none keeps state in scratch memory. A
reload from there waits for every load and store in flight, which the
pipelined kernels never do themselves."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2503_16428_amd import build as B

LLVM = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin")


def test_no_kernel_spills_to_scratch(tmp_path):
    if not os.path.exists(os.path.join(LLVM, "llvm-objdump")):
        pytest.skip("llvm-objdump not available")
    shutil.copy(B.LIB, tmp_path / "lib.so")
    subprocess.run([os.path.join(LLVM, "llvm-objdump"), "--offloading", "lib.so"], cwd=tmp_path,
                   check=True, capture_output=True)
    kernels = {}
    for f in sorted(tmp_path.glob("*gfx950*")):
        notes = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", str(f)], check=True,
                               capture_output=True, text=True).stdout
        for k in notes.split("- .agpr_count:")[1:]:
            kernels[re.search(r"\.name: +(\S+)", k)[1]] = tuple(
                int(re.search(rf"\.{n}: +(\d+)", k)[1])
                for n in ("private_segment_fixed_size", "vgpr_spill_count"))
    assert any("score_partials" in n for n in kernels) and any("attn_kernel" in n for n in kernels)
    assert {n: v for n, v in kernels.items() if v != (0, 0)} == {}
