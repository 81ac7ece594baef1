"""GPU: which kernel a handle below the sizes that are tuned takes (lane-per-node tiles or one round of the
two-step kernel's workgroups), and that its runs equal the one-step kernel's bit for bit: states, totals and flags,
after single steps (which take a kernel of their own beside the two-step one), pairs, an odd count and a captured
graph."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_1009_0254_amd import workloads as W  # noqa: E402

ENV = ("LBF_TILE", "LBF_TILE2", "LBF_STEPS_PER_LAUNCH", "LBF_NODE_TILE")


def replicas(n, nx, ny, **kw):
    return [W.single_phase(nx, ny, kT=1e-5, seed=40 + r, replica=r, **kw) for r in range(n)]


#        replicas, FP32 and FP64: width of the launch's workgroups
CASES = [("56x256^2", replicas(56, 256, 256), 256, 256),
         ("220x128^2", replicas(220, 128, 128), 128, 128),
         ("1000x64^2", replicas(1000, 64, 64), 128, 128),
         ("15x512^2", replicas(15, 512, 512), 512, 512),
         ("2x1400^2", replicas(2, 1400, 1400), 256, 256),
         ("250x16000", replicas(1, 250, 16000), 256, 256),
         ("1800x1900", replicas(1, 1800, 1900), 64, 256),
         ("1000000x3", replicas(1, 1000000, 3), 256, 64),
         ("8x300000", replicas(1, 8, 300000), 128, 128),
         ("2x1024^2", replicas(2, 1024, 1024), 64, 64),
         ("300x9000", replicas(1, 300, 9000), 64, 64),
         ("100000x3", replicas(1, 100000, 3), 64, 64),
         ("correlated", replicas(40, 256, 256) + replicas(14, 256, 256, noise="correlated"), 256, 256)]


@pytest.mark.parametrize("label,cfgs,w32,w64", CASES, ids=[c[0] for c in CASES])
@pytest.mark.parametrize("precision", [2, 0])
def test_choice_and_bits(monkeypatch, label, cfgs, w32, w64, precision):
    from paper_1009_0254_amd import lbfluct as L
    got = []
    some = sorted({0, len(cfgs) // 2, len(cfgs) - 1})
    for env in ({}, {"LBF_TILE": "256,16", "LBF_STEPS_PER_LAUNCH": "1"}):
        for k in ENV:
            monkeypatch.delenv(k, raising=False)
        for k, v in env.items():
            monkeypatch.setenv(k, v)
        print("[gpu-dispatch]", label, "precision", precision, env, file=sys.stderr, flush=True)
        lat = L.Lattice(cfgs, precision=precision)
        if not env:
            width, _, _, steps = lat.lb_tuning()
            assert (width, steps) == (w64 if precision == 0 else w32, 2)
        out = []
        for n in (1, 2, 3, 33):
            lat.step(n)
            out.append(([lat.lb_moments(r) for r in some], lat.lb_status_flags()))
        got.append(out)
        lat.close()
    for (mg, fg), (mr, fr) in zip(*got):
        assert fg == fr
        for (g, tg), (r, tr) in zip(mg, mr):
            assert torch.equal(g, r) and np.array_equal(tg, tr)


def test_tiles_no_taller_than_the_lattice(monkeypatch):
    """A lattice of three rows: two steps in tiles that store those three, not twelve."""
    from paper_1009_0254_amd import lbfluct as L
    for k in ENV:
        monkeypatch.delenv(k, raising=False)
    lat = L.Lattice(replicas(1, 100000, 3), precision="fp32s")
    assert lat.lb_tuning() == (64, 3, 1667, 2)
    lat.close()


@pytest.mark.parametrize("precision,noise", [("fp64", "k0"), ("fp32s", "correlated"), ("fp64", "correlated")])
def test_four_steps_are_refused_without_a_kernel(monkeypatch, precision, noise):
    from paper_1009_0254_amd import lbfluct as L
    for k in ENV:
        monkeypatch.delenv(k, raising=False)
    monkeypatch.setenv("LBF_NODE_TILE", "4,16")
    with pytest.raises(L.LbError) as e:
        L.Lattice(W.single_phase(64, 64, kT=1e-5, seed=1, noise=noise), precision=precision)
    assert e.value.status == L.LB_EINVAL
