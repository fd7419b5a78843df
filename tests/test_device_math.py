"""The device building blocks of physics.h (reconstruction and HLLC flux),
built for the CPU with stand-ins for the hardware's estimates
(tests/device_math), against the oracle's at the ends of their ranges: where
a product of several small or large factors leaves the range of its type
although the result does not."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import oracle
from paper_2305_09163_amd import workloads as W

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2305_09163_amd", "csrc")


@pytest.fixture(scope="module")
def dm(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("device_math") / "device_math.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-ffp-contract=off", "-w", "-shared", "-fPIC",
                    "-I" + os.path.join(HERE, "device_math"), "-I" + CSRC, "-o", lib,
                    os.path.join(HERE, "device_math", "harness.cpp")], check=True)
    return ctypes.CDLL(lib)


def _p(a):
    return a.ctypes.data_as(ctypes.c_void_p)


def uniform_row():
    """The coefficient row of a cell among cells of equal widths: a1, a2
    (times sqrt(13/3)) and the weighted increments at either face in the
    differences of each stencil, then the ideal weights."""
    k = np.sqrt(13.0 / 3.0) / 2.0
    inc = lambda d, t: [d / 6.0 * x for x in t]
    return np.array([-0.5, 1.5, 0.5, 0.5, 1.5, -0.5] + [-k, k] * 3
                    + inc(0.1, (-2, 5)) + inc(0.6, (1, 2)) + inc(0.3, (4, -1))
                    + inc(0.3, (1, -4)) + inc(0.6, (-2, -1)) + inc(0.1, (-5, 2))
                    + [0.1, 0.6, 0.3, 0.3, 0.6, 0.1])


STENCILS = {
    "constant": (3.0, 3.0, 3.0, 3.0, 3.0),
    "smooth": (1.0, 1.1, 1.25, 1.3, 1.28),
    "jump": (1.0, 1.0, 1.0, 1.0e9, 1.0e9),
    "far jump": (1.0, 1.0, 1.0, 1.0, 1.0e9),
    "tails": (0.0, 1.0e-46, 3.0e-46, 2.0e-44, 1.0e-43),
    "huge": (1.0e31, 2.0e31, 2.5e31, 9.0e31, 9.5e31),
}


@pytest.mark.parametrize("eps", [1e-6, 1e-40, 1e-100, 1e-150])
@pytest.mark.parametrize("name", sorted(STENCILS))
def test_weno5_nonuniform_fp64(dm, name, eps):
    """Every stencil whose (eps + beta_r)^2 are FP64 numbers, as the
    definition needs.  Both sides round the differences, a1 and a2 once or
    twice and the weights a few times: 64 roundings of the largest value."""
    s, row = np.array(STENCILS[name]), uniform_row()
    assert dm.dm_coefs() == row.size
    plus, minus = np.empty(1), np.empty(1)
    dm.dm_weno5_nonuniform(_p(row), _p(s), ctypes.c_double(eps), _p(plus), _p(minus))
    ref = oracle.weno5_nonuniform(np.ones(5), s, eps)
    # the face value is a sum of candidates, each within a few of the largest value
    tol = 64 * np.finfo(np.float64).eps * np.abs(s).max()
    assert abs(plus[0] - ref[0]) <= tol and abs(minus[0] - ref[1]) <= tol, (plus, minus, ref)


@pytest.mark.parametrize("order,dtype", [(5, np.float64), (5, np.float32), (3, np.float64), (3, np.float32)])
@pytest.mark.parametrize("eps", [1e-6, 1e-37, 1e-40, 1e-100, 1e-150])
@pytest.mark.parametrize("name", ["constant", "smooth", "jump", "far jump"])
def test_small_eps_on_uniform_cells(dm, name, eps, order, dtype):
    """An epsilon below what the products can hold: differences of FP32 or
    FP64 values of order one are far above its root, or zero."""
    s = np.array(STENCILS[name][:5] if order == 5 else STENCILS[name][1:4], dtype)
    plus, minus = np.empty(1, dtype), np.empty(1, dtype)
    f = getattr(dm, f"dm_weno{order}" + ("" if dtype == np.float64 else "_f"))
    f(_p(s), (ctypes.c_double if dtype == np.float64 else ctypes.c_float)(eps), _p(plus), _p(minus))
    ref = (oracle.weno5 if order == 5 else oracle.weno3)(s.astype(float), eps)
    tol = 64 * np.finfo(dtype).eps * np.abs(s).max()
    assert abs(plus[0] - ref[0]) <= tol and abs(minus[0] - ref[1]) <= tol, (plus, minus, ref)


@pytest.mark.parametrize("uniform", [True, False])
@pytest.mark.parametrize("s", [(1, 1, 1, 1e20, 1e20), (1e20, 1e20, 1, 1, 1), (1, 1, 1, 1, 1e25), (1e25, 1, 1, 1, 1),
                               (1, 1.5, 2, 1e22, 3e22), (3e22, 1e22, 2, 1.5, 1), (1, 1, 1, 2e19, 1), (1, 1.5, 2, 1e9, 1e9),
                               (1, 1.5, 2, 1e13, 1e13), (2e18, 1e18, 2, 1.5, 1)])
def test_weno5_fp32_beside_a_jump(dm, s, uniform):
    """A smooth outer stencil beside differences whose squares overflow FP32:
    the face values are that stencil's, each a few roundings of its own values
    of order one (the jump itself only to its own last place)."""
    s = np.array(s, np.float32)
    plus, minus = np.empty(1, np.float32), np.empty(1, np.float32)
    if uniform:
        dm.dm_weno5_f(_p(s), ctypes.c_float(1e-6), _p(plus), _p(minus))
    else:
        dm.dm_weno5_nonuniform_f(_p(uniform_row()), _p(s), ctypes.c_float(1e-6), _p(plus), _p(minus))
    ref = oracle.weno5(s.astype(float), float(np.float32(1e-6)))[:2]
    assert max(np.abs(ref)) < 10
    for got, want in zip((plus[0], minus[0]), ref):
        assert abs(got - want) <= 32 * np.finfo(np.float32).eps, (got, want)


GAMMA, PI_INF = np.array([4.4, 1.4]), np.array([0.0, 0.0])


def hllc(dm, dtype, wL, wR):
    F, uf = np.empty(5, dtype), np.empty(1, dtype)
    f = dm.dm_hllc if dtype == np.float64 else dm.dm_hllc_f
    bad = f(_p(GAMMA), _p(PI_INF), _p(np.array(wL, dtype)), _p(np.array(wR, dtype)), _p(F), _p(uf))
    spec = W.GridSpec(ndim=1, n=(8,), gamma=tuple(GAMMA), pi_inf=tuple(PI_INF))
    # the oracle's, from the values as rounded to dtype
    ref, uref, st = oracle.hllc(spec, 0, np.array(wL, dtype).astype(float), np.array(wR, dtype).astype(float))
    return (F.astype(float), float(uf[0]), bad), (ref, uref, st)


@pytest.mark.parametrize("dtype,u,p", [(np.float64, 1.0e9, 1.0e-18), (np.float32, 1.0e4, 1.0e-9)])
@pytest.mark.parametrize("sign", [1.0, -1.0])
def test_hllc_supersonic_with_no_fan(dm, dtype, u, p, sign):
    """A sound speed below half a unit in the last place of the velocity: both
    signal speeds round to the velocity, s* is no number, and the flux is that
    of the upwind side."""
    L, R = [0.25, 0.75, sign * u, p, 0.25], [0.5, 1.0, sign * u, 2.0 * p, 0.25]
    (F, uf, bad), (ref, uref, st) = hllc(dm, dtype, L, R)
    assert not bad and st == oracle.OK and uf == uref
    tol = 8 * np.finfo(dtype).eps   # products of three or four factors
    assert (np.abs(F - ref) <= tol * np.abs(ref)).all(), (F, ref)


@pytest.mark.parametrize("dtype,scale", [(np.float64, 2.0 ** -560), (np.float64, 2.0 ** 500), (np.float32, 2.0 ** -80),
                                         (np.float32, 2.0 ** 62), (np.float64, 1.0), (np.float32, 1.0)])
def test_hllc_units(dm, dtype, scale):
    """Densities and pressures whose product leaves the type's range."""
    L, R = [0.25 * scale, 0.75 * scale, 0.5, 3.0 * scale, 0.25], [0.5 * scale, 1.0 * scale, 0.25, 1.5 * scale, 0.5]
    (F, uf, bad), (ref, uref, st) = hllc(dm, dtype, L, R)
    assert not bad and st == oracle.OK
    tol = 16 * np.finfo(dtype).eps   # signal speeds of a few roundings, then products of three or four factors
    assert (np.abs(F - ref) <= tol * np.abs(ref)).all() and abs(uf - uref) <= tol, (F, ref)


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("row,value", [(3, -2.0), (0, -2.0), (3, np.nan), (3, np.inf), (0, np.inf), (0, 0.0)])
def test_hllc_reports_non_physical_sides(dm, dtype, row, value):
    good, side = [0.25, 0.75, 0.5, 3.0, 0.25], [0.25, 0.75, 0.5, 3.0, 0.25]
    side[row] = value
    if value == 0.0:
        side[1] = 0.0   # no density at all
    for L, R in ((good, side), (side, good)):
        F, uf = np.empty(5, dtype), np.empty(1, dtype)
        f = dm.dm_hllc if dtype == np.float64 else dm.dm_hllc_f
        assert f(_p(GAMMA), _p(PI_INF), _p(np.array(L, dtype)), _p(np.array(R, dtype)), _p(F), _p(uf))
