"""GPU: the totals of lb_moments, whichever way they are added up (on the host from pinned memory, or on the
device when a handle has no pinned block), against lb_moments_static (device): bitwise, as the additions and their
order are the same.  Sizes: fewer partial sums than the reduction has lanes, more (its lanes then take several), and
the most there are; and more handles at once than there are pinned blocks.  With a block no call takes memory or
copies, so calls go on while another stream is being captured."""
import ctypes
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_1009_0254_amd import workloads as W  # noqa: E402

GLOBAL = 0     # capture mode: calls that a capture does not allow fail in every thread
BLOCKS = 16    # pinned blocks of the library


def handles(n, cfgs, **kw):
    from paper_1009_0254_amd import lbfluct as L
    out = [L.Lattice(cfgs, **kw) for _ in range(n)]
    for lat in out:
        lat.step(3)
    return out


@pytest.mark.parametrize("precision", [2, 0])
def test_totals_of_every_route_and_size(precision):
    cfgs = [W.single_phase(nx, ny, kT=1e-5, seed=60 + r, replica=r)
            for r, (nx, ny) in enumerate([(40, 24), (300, 300), (512, 511), (700, 600)])]
    lats = handles(BLOCKS + 1, cfgs, precision=precision)
    for lat in (lats[0], lats[-1]):     # with a pinned block (unless other handles live) and without
        for rep, c in enumerate(cfgs):
            print("[gpu-moments]", precision, (c["nx"], c["ny"]), file=sys.stderr, flush=True)
            planes, tot = lat.lb_moments(rep, True)
            again = lat.totals(rep)
            static, ts = lat.lb_moments_static(rep, True)
            assert torch.equal(planes, static)
            assert np.array_equal(tot, ts) and np.array_equal(again, ts)
            # the sums themselves: n additions of FP64 numbers
            m = planes[:3].double()
            sx = 1.0 - 2.0 * (torch.arange(c["nx"], device=m.device) % 2)
            sy = 1.0 - 2.0 * (torch.arange(c["ny"], device=m.device) % 2)
            terms = [m[0], m[1], m[2], m[1] ** 2 + m[2] ** 2, m[1] * sx, m[2] * sy[:, None]]
            for got, t in zip(tot, terms):
                assert abs(got - t.sum().item()) <= 2.3e-16 * t.numel() * t.abs().sum().item()
    for lat in lats:
        lat.close()


def test_calls_during_another_streams_capture():
    """A handle's second call, the first having been made before the capture."""
    from paper_1009_0254_amd import lbfluct as L
    lib = ctypes.CDLL(L.LIB_PATH)      # HIP's capture calls, from the runtime that the library is linked to
    lib.hipStreamBeginCapture.argtypes = [ctypes.c_void_p, ctypes.c_int]
    lib.hipStreamEndCapture.argtypes = [ctypes.c_void_p, ctypes.POINTER(ctypes.c_void_p)]
    lib.hipGraphDestroy.argtypes = [ctypes.c_void_p]
    stream, other = torch.cuda.Stream(), torch.cuda.Stream()
    with torch.cuda.stream(stream):
        lat, = handles(1, [W.single_phase(64, 64, kT=1e-5, seed=5)], precision="fp64")
        want = lat.totals(0)
    torch.cuda.synchronize()
    print("[gpu-moments] capture", file=sys.stderr, flush=True)
    tot = (ctypes.c_double * 6)()
    assert lib.hipStreamBeginCapture(other.cuda_stream, GLOBAL) == 0
    status = L.lib().lb_moments(lat._h, 0, None, tot)
    graph = ctypes.c_void_p()
    ended = lib.hipStreamEndCapture(other.cuda_stream, ctypes.byref(graph))
    lib.hipGetLastError()
    assert (status, ended) == (0, 0)
    assert np.array_equal(np.array(tot[:]), want)
    lib.hipGraphDestroy(graph)
    lat.close()
