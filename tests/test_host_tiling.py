"""The tiles of multi-step launches (csrc/tiling.cpp, no HIP) under the
address and undefined-behaviour sanitizers, driven by
tests/host/tiling_sanitize.cpp on seeded random domains, boundaries and plans:
every node in one tile, every pull of a region in the array and of the
population that the whole domain's pull reads."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_tiles_under_sanitizers(tmp_path):
    exe = str(tmp_path / "tiling_sanitize")
    b = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fno-omit-frame-pointer",
                        "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                        os.path.join(ROOT, "paper_1712_08288_amd", "csrc", "tiling.cpp"),
                        os.path.join(ROOT, "tests", "host", "tiling_sanitize.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert b.returncode == 0, b.stderr[-3000:]
    env = dict(os.environ, ASAN_OPTIONS="verify_asan_link_order=0:detect_leaks=1",
               UBSAN_OPTIONS="print_stacktrace=1")
    r = subprocess.run([exe], capture_output=True, text=True, env=env, timeout=300)
    out = r.stdout + r.stderr
    assert r.returncode == 0 and out.startswith("ok:"), out[-4000:]
