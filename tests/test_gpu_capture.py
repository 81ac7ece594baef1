"""GPU: a synchronous call on a stream under capture is refused (its kernel has not run, so there is
nothing to return).  The runtime leaves that stream invalidated, so what follows runs on another."""
import ctypes
import sys

import numpy as np
import pytest
import torch

sys.path.insert(0, ".")
from paper_1009_0254_amd import lbfluct as L, workloads as W  # noqa: E402

pytestmark = pytest.mark.gpu

RELAXED = 2


def hip():
    """HIP's capture calls, from the runtime that the library itself is linked to."""
    lib = ctypes.CDLL(L.LIB_PATH)
    lib.hipStreamBeginCapture.argtypes = [ctypes.c_void_p, ctypes.c_int]
    lib.hipStreamEndCapture.argtypes = [ctypes.c_void_p, ctypes.POINTER(ctypes.c_void_p)]
    return lib


def sampled(stream):
    with torch.cuda.stream(stream):
        lat = L.Lattice([W.single_phase(64, 64, kT=1e-5, seed=5)], precision="fp64", structure_factor=True)
        lat.lb_step(3)
        lat.lb_structure_factor(L.LB_SK_SAMPLE)
        spectrum, _ = lat.lb_structure_factor(L.LB_SK_READ, 0)
        totals = lat.totals(0)
        stream.synchronize()
    return lat, spectrum, totals


@pytest.mark.parametrize("call", ["moments", "read"])
def test_synchronous_call_under_capture_is_refused(call):
    lib, stream = hip(), torch.cuda.Stream()
    lat, spectrum, totals = sampled(stream)
    print("capture", call, flush=True)
    assert lib.hipStreamBeginCapture(stream.cuda_stream, RELAXED) == 0
    if call == "moments":
        status = L.lib().lb_moments(lat._h, 0, None, (ctypes.c_double * 6)())
    else:
        status = L.lib().lb_structure_factor(lat._h, L.LB_SK_READ, 0, spectrum.data_ptr(), None)
    graph = ctypes.c_void_p()
    lib.hipStreamEndCapture(stream.cuda_stream, ctypes.byref(graph))
    lib.hipGetLastError()   # the refusal's own error, which stays until it is read
    assert status != 0
    other, again, t = sampled(torch.cuda.Stream())
    assert torch.equal(again, spectrum) and np.array_equal(t, totals)
    other.close()
