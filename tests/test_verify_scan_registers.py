"""Registers of the alignment check's scan of all columns (AMD assembly of this
library's own source, cross-compiled for gfx950 on the CPU): for reads of up to
128 bases it keeps 8 wavefronts a SIMD, for up to 256 as many as its LDS allows (4),
which it had before the piece search and loses in one kernel with it."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1711_01177_amd", "csrc")


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not installed")
def test_scan_kernel_registers(tmp_path):
    out = tmp_path / "checker.s"
    subprocess.check_call(
        ["hipcc", "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature",
         "-Xclang", "-packed-fp32-ops", f"-I{os.path.join(ROOT, 'include')}", f"-I{CSRC}",
         "--cuda-device-only", "-S", "-o", str(out), os.path.join(CSRC, "grim_checker.hip")],
        stderr=subprocess.DEVNULL)
    text = out.read_text()
    regs = {int(m.group(1)): int(m.group(2)) for m in re.finditer(
        r"\.name:\s+_ZN4grim18verify_scan_kernelILi(\d)ELb0E.*?\.vgpr_count:\s+(\d+)", text, re.S)}
    assert sorted(regs) == [1, 2, 4, 8]
    for w, limit in ((1, 64), (2, 64), (4, 128), (8, 256)):
        assert regs[w] <= limit, (w, regs[w])
