"""Host: launches of the lane-per-node kernel that have no kernel or no tile are errors, not launches of nothing
(tests/tile_launch_check.cpp, linked with the library's own launch code)."""
import os
import subprocess

import pytest

from paper_1009_0254_amd import build as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1009_0254_amd", "csrc")


def test_launches_without_a_kernel_are_refused(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not found")
    exe = str(tmp_path / "tile")
    flags = [f for f in B.FLAGS if f not in ("-shared", "-O3")] + ["-O1"]
    subprocess.run([hipcc, *flags, "-I", CSRC, "-x", "hip", os.path.join(CSRC, "lb_tile.hip"),
                    os.path.join(ROOT, "tests", "tile_launch_check.cpp"), "-o", exe], check=True, capture_output=True, text=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    print(r.stdout)
    assert r.returncode == 0, r.stdout + r.stderr
