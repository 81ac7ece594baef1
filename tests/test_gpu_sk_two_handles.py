"""GPU: a handle whose S(k) blocks take the most LDS samples after a small one of the same storage was made (the
kernels' LDS limits belong to the process): the same spectra as before it."""
import sys

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_1009_0254_amd import workloads as W  # noqa: E402


@pytest.mark.parametrize("precision", [0, 2])
@pytest.mark.parametrize("shape", [(8192, 16), (16, 16384)], ids=["8192x16", "16x16384"])
def test_large_samples_after_small_is_made(precision, shape):
    from paper_1009_0254_amd import lbfluct as L
    print("[gpu-sk-two]", shape, "precision", precision, file=sys.stderr, flush=True)
    large = L.Lattice(W.single_phase(*shape, kT=1e-5, seed=12), precision=precision, structure_factor=True)
    large.step(4)
    out = []
    for _ in range(2):
        large.lb_structure_factor(L.LB_SK_RESET)
        large.lb_structure_factor(L.LB_SK_SAMPLE)
        out.append((large.lb_structure_factor(L.LB_SK_READ, 0)[0], large.lb_structure_factor(L.LB_SK_SNAPSHOT, 0)))
        small = L.Lattice(W.single_phase(16, 16, kT=1e-5, seed=1), precision=precision, structure_factor=True)
        small.step(1)
        small.lb_structure_factor(L.LB_SK_SAMPLE)
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    small.close()
    large.close()
