"""The decision for all-zero indicator features, which wavefronts without any
difference take from one stored logit, with a network whose every layer and
bias counts: thresholds just below and just above its P(smooth) of zero
features give the all-linear and the all-WENO5 right-hand side, and a single
cell with another volume fraction, density or pressure alone takes the
network's own decisions, as the oracle's."""
import dataclasses
import sys

import numpy as np
import pytest
import torch

import oracle
from oracle import indicator as ind
from parity_util import rhs_err
from paper_2305_09163_amd import mfc
from paper_2305_09163_amd import workloads as W

pytestmark = pytest.mark.gpu

GRIDS = [((20, 18, 16), mfc.MFC_KERNEL_SPLIT), ((20, 18, 16), mfc.MFC_KERNEL_FUSED), ((40, 33), mfc.MFC_KERNEL_FUSED),
         ((300,), mfc.MFC_KERNEL_FUSED)]


def network():
    p = ind.init_params(5)
    rng = np.random.default_rng(55)
    for k in ("b1", "b2", "b3"):
        p[k] = rng.normal(0.0, 0.5, size=p[k].shape)
    p["W3"] = p["W3"] * 4.0
    return ind.unflatten(ind.flatten(p).astype(np.float32).astype(np.float64))


def p_zero(net):
    t = mfc.Trainer(64)
    t.set_params(ind.flatten(net).astype(np.float32))
    return float(t.infer(torch.zeros((64, 16), dtype=torch.int16, device="cuda"))[0])


def state(n, bump=None):
    """Uniform volume fraction, density and pressure, the same bits in every
    cell (powers of two; equal gases, so that the volume fraction does not
    enter the pressure), random velocities; one cell changed in one of them."""
    nd = len(n)
    spec = W.GridSpec(ndim=nd, n=n, gamma=(1.5, 1.5), pi_inf=(0.0, 0.0), weno_eps=1e-6)
    rng = np.random.default_rng(4)
    q = np.zeros(spec.shape)
    q[0], q[1], q[-1] = 2.0 ** -10, 1.0 - 2.0 ** -10, 2.0 ** -2
    u = rng.integers(-32, 33, size=(nd,) + spec.shape[1:]) / 8.0
    at = tuple(s // 2 for s in spec.shape[1:])
    if bump == "rho":
        u[(slice(None),) + at] = 0.0
    q[2:2 + nd] = u
    q[-2] = 2.0 ** 14 + 0.5 * (u ** 2).sum(0)
    if bump:
        row, by = {"alpha": (-1, 2.0 ** -3), "rho": (1, 1.0), "p": (-2, 1024.0)}[bump]
        q[(row,) + at] += by
    return spec, q


def routed(spec, q, kernel, precision, net, tau):
    s = mfc.Solver(spec, precision=precision, recon=mfc.MFC_RECON_LEARNED, kernel=kernel)
    s.set_indicator(ind.flatten(net).astype(np.float32), tau)
    d = s.upload(q)
    s.fill_ghosts(d)
    r = s.rhs(d)
    s.check()
    return r


@pytest.mark.parametrize("precision", [mfc.MFC_FP64, mfc.MFC_FP32_MIXED])
@pytest.mark.parametrize("n,kernel", GRIDS)
def test_threshold_at_the_zero_features(n, kernel, precision):
    print(f"[zero logit] {n} kernel {kernel} precision {precision}", file=sys.stderr, flush=True)
    net = network()
    spec, q = state(n)
    p0 = p_zero(net)
    assert 0.1 < p0 < 0.9
    # the FP32 logit, P and threshold differ by a few roundings of order one
    linear, weno = (routed(spec, q, kernel, precision, net, t) for t in (0.0, 1.0))
    assert not torch.equal(linear, weno)
    assert torch.equal(routed(spec, q, kernel, precision, net, p0 - 1e-5), linear)
    assert torch.equal(routed(spec, q, kernel, precision, net, p0 + 1e-5), weno)


@pytest.mark.parametrize("precision", [mfc.MFC_FP64, mfc.MFC_FP32_MIXED])
@pytest.mark.parametrize("bump", ["alpha", "rho", "p"])
@pytest.mark.parametrize("n,kernel", GRIDS)
def test_one_cell_that_differs(n, kernel, bump, precision):
    print(f"[zero logit] {n} kernel {kernel} precision {precision} {bump}", file=sys.stderr, flush=True)
    net = network()
    spec, q = state(n, bump)
    q = oracle.fill_ghosts(spec, q)
    P = ind.smooth_probability(spec, q, net)
    Pv = P[~np.isnan(P)]
    p0 = p_zero(net)
    far = Pv[np.argmax(np.abs(Pv - p0))]
    tau = float(0.5 * (p0 + far))
    # both routes are taken, and no decision is close
    assert np.abs(Pv - tau).min() > 1e-3 and (Pv > tau).any() and (Pv < tau).any()
    ref, st, _ = ind.rhs_learned(spec, q, net, tau)
    assert st == oracle.OK
    # FP64 as every routed right-hand side; FP32: a few hundred roundings
    bar = 1e-12 if precision == mfc.MFC_FP64 else 1e-5
    other, st, _ = ind.rhs_learned(spec, q, net, 0.0 if p0 > tau else 1.0)   # the bump ignored
    assert st == oracle.OK and rhs_err(other, ref, q, spec).max() > 10 * bar
    got = routed(spec, q, kernel, precision, net, tau).double().cpu().numpy()
    err = rhs_err(got, ref, q, spec)
    assert err.max() <= bar, err


@pytest.mark.parametrize("n,kernel", GRIDS)
def test_small_weno_eps_in_fp32(n, kernel):
    """The floor of the features' divisor, sqrt(weno_eps), below FP32's normal
    numbers: zero differences still give zero features."""
    print(f"[zero logit] {n} kernel {kernel} eps 1e-80", file=sys.stderr, flush=True)
    net = network()
    spec, q = state(n)
    spec = dataclasses.replace(spec, weno_eps=1e-80)
    p0 = p_zero(net)
    linear = routed(state(n)[0], q, kernel, mfc.MFC_FP32_MIXED, net, 0.0)   # no epsilon in it
    assert torch.equal(routed(spec, q, kernel, mfc.MFC_FP32_MIXED, net, p0 - 1e-5), linear)
