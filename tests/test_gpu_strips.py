"""GPU: the two-step kernel in strips of every stored width (bx - 6 columns, or in FP32 a multiple of 64
bytes) against the one-step kernel on the same runs.  Both apply the same expressions in the same order, so
states, totals and flags are equal bit for bit.  Widths: one column over a workgroup and over a strip, rows of a
multiple of 64 bytes and not, the shorter strips' own case (1024, and 4096 in a lattice beyond the last-level cache)
and those where they would cost one more strip (481, 1000, 1008)."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_1009_0254_amd import workloads as W  # noqa: E402

#        nx, ny, strips of 256 and of 512 lanes: FP32, FP64
STRIPS = [(257, 24, 2, 1, 2, 1), (481, 24, 2, 1, 2, 1), (513, 24, 3, 2, 3, 2), (1000, 24, 4, 2, 4, 2),
          (1008, 24, 5, 2, 5, 2), (1024, 24, 5, 3, 5, 3), (2000, 24, 8, 4, 8, 4), (4096, 24, 17, 9, 17, 9),
          (4096, 1024, 18, 9, 17, 9)]


@pytest.mark.parametrize("precision", [2, 0, 1])
@pytest.mark.parametrize("nx,ny,s256,s512,d256,d512", STRIPS, ids=["%dx%d" % s[:2] for s in STRIPS])
def test_strips_bitwise(monkeypatch, nx, ny, s256, s512, d256, d512, precision):
    from paper_1009_0254_amd import lbfluct as L
    cfg = W.single_phase(nx, ny, kT=1e-5, seed=nx)
    got = []
    for env in ({"LBF_TILE": "256,16", "LBF_STEPS_PER_LAUNCH": "1"}, {"LBF_TILE2": "256,12"}, {"LBF_TILE2": "512,12"}):
        for k in ("LBF_TILE", "LBF_TILE2", "LBF_STEPS_PER_LAUNCH", "LBF_NODE_TILE"):
            monkeypatch.delenv(k, raising=False)
        for k, v in env.items():
            monkeypatch.setenv(k, v)
        print("[gpu-strips]", nx, "precision", precision, env, file=sys.stderr, flush=True)
        lat = L.Lattice(cfg, precision=precision)
        width, _, workgroups, steps = lat.lb_tuning()
        if steps == 2:
            strips = {256: (d256, s256), 512: (d512, s512)}[width][precision != 0]
            assert workgroups == -(-ny // 12) * strips
        lat.step(37)
        got.append((lat.lb_moments(0), lat.lb_status_flags()))
        lat.close()
    for (m, tot), flags in got[1:]:
        assert torch.equal(m, got[0][0][0]) and np.array_equal(tot, got[0][0][1]) and flags == got[0][1]
