"""GPU: the FP64 reciprocal, quotient and square roots of lb_rng.h as the device computes them (seed
and fma residuals; the host build of the same header takes / and sqrt instead), and ln u, sin and cos of 2 pi u
at all 2^21 Box-Muller arguments, against long double.  Bounds: Newton's iteration from the hardware's 2^-24
leaves 2^-46, and the residual formed with fma rounds once, so 0.51 ulp for the four helpers; for ln, sin and cos
the bound that the host build is held to over the same arguments (5e-16 relative), and the host build's bits:
only the quotient differs between the two, and a value within 2^-40 ulp of the exact one rounds as it does."""
import sys

import numpy as np
import pytest

sys.path.insert(0, ".")
torch = pytest.importorskip("torch")

import device_math as M  # noqa: E402

pytestmark = pytest.mark.gpu


def device(what, v, a=None):
    lib = M.lib()
    v = np.ascontiguousarray(v, dtype=np.float64)
    a = np.zeros_like(v) if a is None else np.ascontiguousarray(a, dtype=np.float64)
    dv, da = torch.from_numpy(v).cuda(), torch.from_numpy(a).cuda()
    out = torch.empty_like(dv)
    assert lib.device_eval(what, da.data_ptr(), dv.data_ptr(), out.data_ptr(), len(v),
                           torch.cuda.current_stream().cuda_stream) == 0
    return out.cpu().numpy()


def host(what, v, a=None):
    out = np.empty_like(v)
    a = np.zeros_like(v) if a is None else a
    M.lib().host_eval(what, a.ctypes.data, v.ctypes.data, out.ctypes.data, len(v))
    return out


def ulps(got, want):
    """|got - want| in units of the last place of the wanted value"""
    return np.abs((got.astype(np.longdouble) - want) / np.spacing(np.abs(want.astype(np.float64))))


def arguments(lo, hi, n=1 << 20):
    """logarithmically uniform over [2^lo, 2^hi], and every mantissa region near 1"""
    rng = np.random.default_rng(5)
    v = np.exp2(rng.uniform(lo, hi, n)) * rng.uniform(1, 2, n)
    return np.concatenate([v, 1 + np.arange(-2048, 2048) * 2.0 ** -53, rng.uniform(0.25, 4, n)])


def test_transcendentals_over_every_argument():
    b = np.arange(1 << 21, dtype=np.float64)
    u = (b.astype(np.longdouble) + np.longdouble(0.5)) / 2097152
    pi = np.arctan2(np.longdouble(0), np.longdouble(-1))
    k = np.rint(4 * u)      # quarter turns, taken off exactly
    th = 2 * pi * (u - k / 4)
    s, c, q = np.sin(th), np.cos(th), k.astype(int) & 3
    want = {M.LN: np.log(u), M.SIN: np.choose(q, [s, c, -s, -c]), M.COS: np.choose(q, [c, -s, -c, s])}
    for what, w in want.items():
        got = device(what, b)
        err = np.abs((got - w) / w).max()
        print("device math", what, "relative error", float(err), "off the host build:",
              int((got != host(what, b)).sum()), flush=True)
        assert err < 5e-16
        assert np.array_equal(got, host(what, b))


def test_reciprocal():
    v = arguments(-1021, 1020)
    v = np.concatenate([v, -v])
    e = ulps(device(M.RCP, v), 1 / v.astype(np.longdouble)).max()
    print("device math rcp ulp", float(e), "not as the host's", int((device(M.RCP, v) != 1 / v).sum()), flush=True)
    assert e < 0.51
    got = device(M.RCP, np.array([0.0, -0.0, np.inf, -np.inf, np.nan]))
    assert got[0] == np.inf and got[1] == -np.inf and got[2] == 0 and got[3] == 0 and np.isnan(got[4])


def test_quotient():
    v = arguments(-400, 400)
    a = np.random.default_rng(6).permutation(arguments(-400, 400))
    a[::2] *= -1
    e = ulps(device(M.DIV, v, a), a.astype(np.longdouble) / v).max()
    print("device math div ulp", float(e), "not as the host's", int((device(M.DIV, v, a) != a / v).sum()), flush=True)
    assert e < 0.51
    assert (device(M.DIV, v, np.zeros_like(v)) == 0).all()


def test_square_root():
    v = np.concatenate([arguments(-960, 1020), np.arange(1, 4097, dtype=np.float64) ** 2])
    for what in (M.SQRT, M.ROOT):
        e = ulps(device(what, v), np.sqrt(v.astype(np.longdouble))).max()
        print("device math sqrt", what, "ulp", float(e), "not as the host's",
              int((device(what, v) != np.sqrt(v)).sum()), flush=True)
        assert e < 0.51
    # 1 / r of the rounded root r
    r = device(M.ROOT, v)
    e = ulps(device(M.RROOT, v), 1 / r.astype(np.longdouble)).max()
    print("device math 1 / sqrt ulp", float(e), "not as the host's", int((device(M.RROOT, v) != 1 / r).sum()), flush=True)
    assert e < 0.51
    # where the last residual rounds away: Newton's step from the estimate
    w = np.concatenate([np.exp2(np.random.default_rng(7).uniform(-1074, -960, 1 << 16)), [2.0 ** -1074]])
    want = np.sqrt(w.astype(np.longdouble))
    assert (np.abs((device(M.SQRT, w) - want) / want) < 2.0 ** -44).all()
    assert device(M.SQRT, np.array([0.0]))[0] == 0 and np.isnan(device(M.SQRT, np.array([np.nan]))[0])
