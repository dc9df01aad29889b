"""The compile-time value bounds of the transforms' passes (CPU)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2603_22437_amd", "csrc")


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not available")
def test_moddown_entry_bounds(tmp_path):
    """ModDown's forward pass is compiled for at least the values it is given,
    on every path of the basis conversion before it."""
    exe = tmp_path / "pass_bounds_test"
    subprocess.run(["hipcc", "-x", "hip", "--offload-host-only", "-std=c++17", "-O0",
                    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                    os.path.join(ROOT, "tests", "cpp", "pass_bounds_test.cpp"), "-o", str(exe)],
                   check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "all checks passed" in r.stdout
