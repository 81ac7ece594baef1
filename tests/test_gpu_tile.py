"""GPU: the kernel of small and middle-sized lattices (a lane per node, tiles of 64 columns, one,
two or four steps per launch) against the one-step kernel that marches strips down their rows, on
the same runs.  Both apply the same expressions to every node in the same order, so the states, the
totals and the flags are equal bit for bit, whatever the tiling: no tolerance.

Sizes where the tiling can go wrong: rows of one lane less, as many and one more than a tile's 64
columns and the 60 (two steps) or 52 (four) that it stores, last bands and strips of one row or
column, a lattice lower than a tile's halo (rows wrap more than once), several replicas of mixed
widths in one launch, every storage and noise.
"""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_1009_0254_amd import workloads as W  # noqa: E402

CASES = [
    ("3x5", [W.single_phase(3, 5, kT=1e-5, seed=2)]),
    ("53x61", [W.single_phase(53, 61, kT=1e-5, seed=3, noise="diagonal")]),
    ("63x13", [W.single_phase(63, 13, kT=1e-5, seed=4)]),
    ("64x33", [W.slab(64, 33, kT=1e-6, seed=5)]),
    ("65x21", [W.single_phase(65, 21, kT=1e-5, seed=6)]),
    ("105x40", [W.wave(W.single_phase(105, 40, kT=0), 1, 2, 1e-3, 0, 1e-4)]),
    ("121x4", [W.single_phase(121, 4, kT=1e-5, seed=7)]),
    ("1021x37", [W.spinodal(1021, 37, kT=1e-6, seed=8)]),
    ("mixed", [W.single_phase(128, 40, kT=1e-5, seed=21, replica=0),
               W.single_phase(64, 24, kT=2e-5, seed=22, replica=1),
               W.single_phase(600, 18, kT=1e-5, seed=24, replica=3),
               W.wave(W.single_phase(3, 9, kT=0), 1, 1, 1e-4, 0, 1e-4),
               W.slab(40, 64, kT=1e-6, seed=25, replica=5)]),
    ("correlated", [dict(W.correlated_sec5a(64, 32, kT=1e-6, seed=31), replica=0),
                    W.single_phase(100, 36, kT=1e-5, seed=32, replica=1),
                    dict(W.correlated_sec5a(256, 16, kT=1e-6, seed=33), replica=2)]),
]
CASES += [("correlated-" + f"{nx}x{ny}", [W.correlated_sec5a(nx, ny, kT=1e-6, seed=34)])   # four steps' fields at once
          for nx, ny in ((4, 4), (8, 8), (128, 32))]                              # (from 64 nodes on, FP32)
TILES = ["1,4", "1,16", "2,5", "2,8", "2,16", "4,13", "4,16", None]   # None: the handle's own choice


@pytest.mark.parametrize("label,cfgs", CASES, ids=[c[0] for c in CASES])
@pytest.mark.parametrize("precision", [2, 0, 1])
def test_node_tiles_bitwise(monkeypatch, label, cfgs, precision):
    from paper_1009_0254_amd import lbfluct as L

    def run(env):
        for k in ("LBF_TILE", "LBF_TILE2", "LBF_STEPS_PER_LAUNCH", "LBF_NODE_TILE"):
            monkeypatch.delenv(k, raising=False)
        for k, v in env.items():
            monkeypatch.setenv(k, v)
        lat = L.Lattice(cfgs, precision=precision)
        steps, out = lat.lb_tuning()[3], []
        for n in (1, 2, 7, 64):   # single steps, pairs, a remainder, the captured graph
            lat.step(n)
            out.append(([lat.lb_moments(r) for r in range(len(cfgs))], lat.lb_status_flags()))
        lat.close()
        return steps, out

    _, ref = run({"LBF_TILE": "256,16", "LBF_STEPS_PER_LAUNCH": "1"})
    for tile in TILES:
        if tile and tile[0] == "4" and (precision == 0 or label.startswith("correlated")):
            continue   # four steps: FP32 without correlated noise only
        print("[gpu-tile]", label, "precision", precision, "tile", tile, file=sys.stderr, flush=True)
        steps, got = run({"LBF_NODE_TILE": tile} if tile else {})
        assert tile is None or steps == int(tile[0])
        for (mg, fg), (mr, fr) in zip(got, ref):
            assert fg == fr
            for (g, tg), (r, tr) in zip(mg, mr):
                assert torch.equal(g, r) and np.array_equal(tg, tr), tile


@pytest.mark.parametrize("tile", ["2,4", "4,12", "1,17", "3,16", "0,8"])
def test_impossible_node_tiles_are_refused(monkeypatch, tile):
    """Shapes that lose all their rows, are taller than a workgroup or have no kernel."""
    from paper_1009_0254_amd import lbfluct as L
    monkeypatch.setenv("LBF_NODE_TILE", tile)
    with pytest.raises(L.LbError):
        L.Lattice(W.single_phase(64, 64, kT=1e-5, seed=1), precision="fp32s")


@pytest.mark.parametrize("shape", [(1700, 1600), (5200, 520), (300, 9000)], ids=["1700x1600", "5200x520", "300x9000"])
@pytest.mark.parametrize("precision", [2, 0])
def test_middle_sizes_bitwise(monkeypatch, shape, precision):
    """2.7 million nodes, about where a lattice goes from the lane-per-node tiles to one round of the
    two-step kernel's strips (not when a strip would be mostly empty)."""
    from paper_1009_0254_amd import lbfluct as L
    cfg = W.single_phase(*shape, kT=1e-5, seed=9)
    got = []
    for env in ({}, {"LBF_TILE": "256,16", "LBF_STEPS_PER_LAUNCH": "1"}):
        for k in ("LBF_TILE", "LBF_TILE2", "LBF_STEPS_PER_LAUNCH", "LBF_NODE_TILE"):
            monkeypatch.delenv(k, raising=False)
        for k, v in env.items():
            monkeypatch.setenv(k, v)
        lat = L.Lattice(cfg, precision=precision)
        lat.step(35)
        got.append(lat.lb_moments(0)[0])
        lat.close()
    assert torch.equal(*got)
