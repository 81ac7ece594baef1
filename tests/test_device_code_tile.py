"""The device code of the lane-per-node kernel as the compiler emits it (host only): no packed FP32
instructions, no waterfall loops around its row loads, no scratch."""
from test_device_code import CSRC, HIPCC, ROOT, kernel_meta, kernels, pytestmark, waterfall_loops  # noqa: F401

import os
import re
import subprocess

from paper_1009_0254_amd import build as B


def test_tile_kernels(tmp_path):
    flags = [f for f in B.FLAGS if f not in ("-shared", "-fPIC")]
    s = str(tmp_path / "tile.s")
    subprocess.run([HIPCC, *flags, "--cuda-device-only", "-S", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                    os.path.join(CSRC, "lb_tile.hip"), "-o", s], check=True, capture_output=True, text=True)
    text = open(s).read()
    assert not re.findall(r"\bv_pk_(?:add|mul|fma)_f32\b", text)
    ks = [(n, b) for n, b in kernels(text) if n.startswith("_ZN3lbf6k_tile")]
    assert len(ks) >= 12
    for name, body in ks:
        assert waterfall_loops(body) == 0, name
        assert kernel_meta(text, name, "amdhsa_private_segment_fixed_size") == 0, name
