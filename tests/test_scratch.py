"""Host logic of optional device scratch (no GPU): when it cannot grow, what a
context holds for its other calls stays.  A small host program compiled
against the library's internal header."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_0707_0438_amd", "csrc")


@pytest.mark.timeout(300)
def test_failed_growth_keeps_the_buffer(tmp_path):
    from paper_0707_0438_amd import build
    exe = str(tmp_path / "scratch")
    cmd = [build.hipcc(), "-O2", "-std=c++17", "-x", "hip", f"--offload-arch={build.ARCH}",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-Wno-unused-command-line-argument", "-I", CSRC,
           os.path.join(ROOT, "tests", "host", "scratch.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    assert subprocess.run([exe], timeout=240).returncode == 0
