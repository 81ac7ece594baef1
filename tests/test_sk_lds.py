"""Host: the dynamic LDS limits of the S(k) kernels cover every lattice, whichever handle set them last
(tests/sk_lds_check.cpp, linked with the library's own launch code)."""
import os
import subprocess

import pytest

from paper_1009_0254_amd import build as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1009_0254_amd", "csrc")


def test_limits_cover_every_lattice(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not found")
    exe = str(tmp_path / "sk_lds")
    flags = [f for f in B.FLAGS if f not in ("-shared", "-O3")] + ["-O1"]
    subprocess.run([hipcc, *flags, "-I", CSRC, "-x", "hip", os.path.join(CSRC, "lb_sk.hip"),
                    os.path.join(ROOT, "tests", "sk_lds_check.cpp"), "-o", exe], check=True, capture_output=True, text=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    print(r.stdout)
    assert r.returncode == 0, r.stdout + r.stderr
