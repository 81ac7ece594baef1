"""GPU: the structure factor of one sample against numpy's transforms of the oracle's moments, at the
shapes where the sampler's blocks change form: a lattice whose columns all fit one block beside the
folded Nyquist column (4 x 4, 8 x 64, 64 x 8), blocks cut for want of work (64 x 64, 256 x 32) and not
(the ensembles, which also take the separate reference kernel), whole columns of 1024 and 2048 points,
register-cached and uncached rows (2048, 4096).

Tolerances as derived for the sampler elsewhere: FP64 1e-10 + 16 eps log2(n) n / sqrt(n S_max) of S_max;
FP32 storage 1e-4 of S_max."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import oracle as O  # noqa: E402
from paper_1009_0254_amd import workloads as W  # noqa: E402


def power(m):
    n = m.shape[1] * m.shape[2]
    return np.abs(np.fft.rfft2(m, axes=(1, 2))) ** 2 / n


def check(got, cfg, moments, precision):
    want = power(moments)
    n = cfg["nx"] * cfg["ny"]
    for a in range(9):
        top = want[a].max()
        tol = 1e-10 + 16 * 2.2e-16 * np.log2(n) * n / np.sqrt(n * top) if precision == 0 else 1e-4
        err = np.abs(got[a] - want[a]).max() / top
        assert err < tol, (cfg["nx"], cfg["ny"], a, err, tol)


SHAPES = [(4, 4), (8, 64), (64, 8), (64, 64), (256, 32), (2048, 16), (4096, 8), (16, 1024), (64, 2048)]


@pytest.mark.parametrize("shape", SHAPES, ids=[f"{a}x{b}" for a, b in SHAPES])
@pytest.mark.parametrize("precision", [0, 2])
def test_sample_of_one_lattice(precision, shape):
    from paper_1009_0254_amd import lbfluct as L
    print("[gpu-sk]", shape, "precision", precision, file=sys.stderr, flush=True)
    cfg = W.single_phase(*shape, kT=1e-5, seed=12)
    lat = L.Lattice(cfg, precision=precision, structure_factor=True)
    lat.step(6)
    lat.lb_structure_factor(L.LB_SK_SAMPLE, -1)
    got, count = lat.lb_structure_factor(L.LB_SK_READ, 0)
    moments = lat.moments() if precision == 2 else None
    lat.close()
    assert count == 1
    if precision == 0:
        o = O.Oracle(cfg)
        o.step(6)
        moments = o.moments()
    check(got.cpu().numpy(), cfg, moments, precision)


@pytest.mark.parametrize("precision", [0, 2])
def test_sample_of_an_ensemble_that_fills_the_chip(precision):
    from paper_1009_0254_amd import lbfluct as L
    sizes = [(128, 128)] * 70 + [(256, 256)] * 4 + [(512, 64), (64, 512), (16, 8)]
    cfgs = [W.single_phase(nx, ny, kT=1e-5, seed=50 + r, replica=r) for r, (nx, ny) in enumerate(sizes)]
    lat = L.Lattice(cfgs, precision=precision, structure_factor=True)
    lat.step(3)
    lat.lb_structure_factor(L.LB_SK_SAMPLE, -1)
    for r in (0, 69, 70, 74, 75, 76):
        got, _ = lat.lb_structure_factor(L.LB_SK_READ, r)
        check(got.cpu().numpy(), cfgs[r], lat.moments(r), precision)
    lat.close()
