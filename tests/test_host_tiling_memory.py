"""The tiles' link tables (csrc/tiling.cpp, no HIP) without memory, driven by
tests/host/tiling_memory.cpp: a table that cannot be had is reported, so that
the handle takes single steps; no exception leaves."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_tile_links_without_memory(tmp_path):
    exe = str(tmp_path / "tiling_memory")
    b = subprocess.run(["g++", "-std=c++17", "-O1",
                        os.path.join(ROOT, "paper_1712_08288_amd", "csrc", "tiling.cpp"),
                        os.path.join(ROOT, "tests", "host", "tiling_memory.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert b.returncode == 0, b.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.startswith("ok:"), (r.returncode, r.stdout + r.stderr)
