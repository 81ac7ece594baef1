"""GPU: the radially binned density snapshot against the oracle's, on the same moments, at the shapes where the
shell sums change form: lanes along ky for tall planes (16 and 4 of them), along kx for wide and square ones, and
two passes over the columns for large planes or very few shells.  Tolerance as for the sample: FP64 1e-10 +
16 eps log2(n) n / sqrt(n S_max) of the largest mode, FP32 storage 1e-4; the counts are whole numbers."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import oracle as O  # noqa: E402
from paper_1009_0254_amd import workloads as W  # noqa: E402

SHAPES = [(4, 64), (16, 4096), (64, 512), (512, 1024), (4, 8), (8, 8), (512, 512), (1024, 64), (4096, 4), (2048, 2048)]


@pytest.mark.parametrize("shape", SHAPES, ids=[f"{a}x{b}" for a, b in SHAPES])
@pytest.mark.parametrize("precision", [0, 2])
def test_snapshot(precision, shape):
    from paper_1009_0254_amd import lbfluct as L
    print("[gpu-snapshot]", shape, "precision", precision, file=sys.stderr, flush=True)
    lat = L.Lattice(W.spinodal(*shape, kT=1e-6, seed=14), precision=precision, structure_factor=True)
    lat.step(5)
    got = lat.lb_structure_factor(L.LB_SK_SNAPSHOT, 0).cpu().numpy()
    rho = lat.moments()[0]
    lat.close()
    mean, counts = O.radial_spectrum(rho)
    n = rho.size
    top = (np.abs(np.fft.rfft2(rho)) ** 2 / n).max()   # k = 0 included: its leakage is what FP64 rounding allows
    off = np.abs(np.fft.rfft2(rho - rho.mean())) ** 2 / n
    tol = (1e-10 * off.max() + 16 * 2.2e-16 * np.log2(n) * np.sqrt(top * off.max())) if precision == 0 else 1e-4 * off.max()
    assert np.array_equal(got[1], counts)
    assert np.abs(got[0] - mean).max() < tol
