"""GPU: FP64 noise whose variances lie below the normal range.  From rest one step adds noise proportional
to sqrt(kT) to modes 4 to 9, and the model's other terms vanish beside it, so their spectra over kT are those
of any other small kT.  (The stored deviations carry such noise; S(k) off k = 0 is formed from them alone.)
Tolerance: a variance below 2^-1022 is a multiple of 2^-1074, so with 3 kT = 3e-309 the smallest -2 ln u
(4.8e-7) leaves an absolute error of 2^-1075 / (2 sqrt(1.4e-315)) = 3.3e-167 in a normal, 6e-13 of
sqrt(3 kT); a Fourier sum of 512 of them, squared, stays within 1e-10 of the spectrum's mean."""
import sys

import pytest

sys.path.insert(0, ".")
from paper_1009_0254_amd import workloads as W  # noqa: E402

pytestmark = pytest.mark.gpu

TINY, SMALL = 1e-309, 1e-250


@pytest.mark.parametrize("noise", ["k0", "correlated"])
def test_spectra_scale_with_a_tiny_temperature(noise):
    from paper_1009_0254_amd import lbfluct as L
    out = []
    for kT in (TINY, SMALL):
        lat = L.Lattice(W.single_phase(32, 16, kT=kT, seed=9, noise=noise), precision="fp64", structure_factor=True)
        lat.step(1)
        lat.lb_structure_factor(L.LB_SK_SAMPLE)
        s, _ = lat.lb_structure_factor(L.LB_SK_READ, 0)
        flags, _ = lat.lb_status_flags()
        lat.close()
        assert flags == 0
        out.append(s[3:].flatten(1)[:, 1:].cpu() / kT)      # modes 4 to 9 off k = 0
    mean = out[1].mean(dim=1)
    err = (out[0] - out[1]).abs().max(dim=1).values / mean
    print("tiny noise", noise, mean, err, flush=True)
    assert (mean[1:5] > 1e-3).all()
    assert (err[1:5] < 1e-10).all()
    if noise == "k0":
        assert (err < 1e-10).all()
