"""Loads in flight of the compiled bin-window kernel (AMD assembly of this
library's own source, cross-compiled for gfx950 on the CPU).

A thread adds 16 tokens' row words at a time, and what a window costs is the
latency of those loads: each instantiation's loops, for windows that start on a
row word (one word a token) and anywhere else (two), ask for all 16 before the
first wait."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1711_01177_amd", "csrc")


def loads_before_wait(body, width):
    """Longest run of row loads of `width` dwords with no wait on memory between."""
    op = re.compile(r"\b(buffer|global)_load_dword" + ("x%d" % width if width > 1 else "") + r"\s")
    best = run = 0
    for line in body:
        if op.search(line):
            run += 1
            best = max(best, run)
        elif "vmcnt" in line or line.startswith(".LBB"):
            run = 0
    return best


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not installed")
def test_sixteen_rows_in_flight(tmp_path):
    out = tmp_path / "window.s"
    subprocess.check_call(
        ["hipcc", "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature",
         "-Xclang", "-packed-fp32-ops", f"-I{os.path.join(ROOT, 'include')}", f"-I{CSRC}",
         "--cuda-device-only", "-S", "-o", str(out), os.path.join(CSRC, "grim_window.hip")],
        stderr=subprocess.DEVNULL)
    lines = out.read_text().splitlines()
    starts = [i for i, l in enumerate(lines) if re.match(r"^_Z\S*window_kernel\S*:", l)]
    assert len(starts) == 16     # q = 4..7, 8 or 16 planes, 32- or 64-bit row offsets
    for a in starts:
        b = next(i for i in range(a, len(lines)) if lines[i].startswith(".Lfunc_end"))
        for width in (1, 2):
            n = loads_before_wait(lines[a:b], width)
            assert n >= 16, (lines[a].split(":")[0], width, n)
