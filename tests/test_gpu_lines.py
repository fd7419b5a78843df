"""Whole-step 1D kernels at the edges of their forms: one workgroup (256, 512
and 1024 threads, more steps than one launch takes) and pieces of 238 cells
(odd and even step counts, which end in different buffers; more pieces than a
step reduces wave speeds for itself).  Against the oracle, the stage-by-stage
path (taken while kernel timing is on) and the ghost cells a fill leaves."""
import dataclasses
import sys

import numpy as np
import pytest
import torch

import oracle
from parity_util import rel_linf, rounding_spread_run, step_bar
from paper_2305_09163_amd import mfc
from paper_2305_09163_amd import workloads as W

pytestmark = pytest.mark.gpu


def faces(n):
    s = np.arange(n + 1) / n
    return s - 0.05 * np.tanh((s - 0.5) / 0.1) + 0.05 * np.tanh(-5.0) * (1.0 - 2.0 * s)


def run(spec, q0, steps, recon=mfc.MFC_RECON_WENO5, precision=mfc.MFC_FP64, stages=False, single=False):
    s = mfc.Solver(spec, recon=recon, precision=precision)
    if stages:
        mfc.mfc_set_kernel_timing(s.h, True)
    q = s.upload(q0)
    if single:
        for _ in range(steps):
            s.step(q, cfl=0.4)
    else:
        s.run(q, steps, cfl=0.4)
    s.check()
    return q.cpu().numpy(), s.time()


@pytest.mark.parametrize("n,steps", [(3, 2), (62, 5), (254, 3), (255, 3), (400, 70), (510, 2), (511, 2), (511, 5),
                                     (1022, 1), (1023, 1), (1023, 2), (1428, 3), (3001, 4)])
@pytest.mark.parametrize("bc", [0, 1])
def test_lines(n, steps, bc):
    spec, w = W.shock_tube_1d(n)
    spec = dataclasses.replace(spec, bc=(bc,) * 6)
    print(f"[lines] {n} cells {steps} steps bc {bc}", file=sys.stderr, flush=True)
    q0 = oracle.prim_to_cons_field(spec, w)
    qn, _, st = oracle.run(spec, q0, steps, cfl=0.4)
    if st != oracle.OK:   # three periodic cells of water against air leave the physical states: both say so
        with pytest.raises(mfc.MfcError):
            run(spec, q0, steps)
        return
    q, t = run(spec, q0, steps)
    # 1e-12 per variable, or twice the oracle's own rounding-order spread over the same run
    bar = step_bar(rounding_spread_run(spec, q0, steps, cfl=0.4, norm="linf"))
    err = rel_linf(q, qn, spec)
    assert (err <= bar).all(), (err, bar)
    p, tp = run(spec, q0, steps, stages=True)
    # step sizes differ by the rounding of the states alone
    assert abs(t[0] - tp[0]) <= 1e-10 * tp[0]
    assert (rel_linf(q, p, spec) <= 2.0 * bar).all()
    # ghost cells: the fill of the last step's start, from the same states
    g, tg = run(spec, q0, steps, single=True)
    I = (slice(None),) + spec.interior[1:]
    assert np.array_equal(g[I], q[I]) or (rel_linf(g, q, spec) <= 2.0 * bar).all()
    before = run(spec, q0, steps - 1)[0] if steps > 1 else q0
    s = mfc.Solver(spec)
    b = s.upload(before)
    s.fill_ghosts(b)
    b, k = b.cpu().numpy(), 3
    for v in range(q.shape[0]):
        scale = np.abs(b[v]).max()
        assert np.abs(q[v, 0, 0, :k] - b[v, 0, 0, :k]).max() <= 1e-10 * scale
        assert np.abs(q[v, 0, 0, -k:] - b[v, 0, 0, -k:]).max() <= 1e-10 * scale


@pytest.mark.parametrize("form", ["weno3", "first", "stretched", "kapila"])
@pytest.mark.parametrize("n,bc", [(400, 0), (900, 0), (900, 1)])
@pytest.mark.parametrize("precision", [mfc.MFC_FP64, mfc.MFC_FP32_MIXED])
def test_forms(form, n, bc, precision):
    spec, w = W.shock_tube_1d(n)
    over = {"bc": (bc,) * 6}
    if form == "stretched":
        over["faces"] = (faces(n), None, None)
    if form == "kapila":
        over["model"] = 1
    spec = dataclasses.replace(spec, **over)
    print(f"[lines] {form} {n} bc {bc} precision {precision}", file=sys.stderr, flush=True)
    recon = {"weno3": mfc.MFC_RECON_WENO3, "first": mfc.MFC_RECON_FIRST_ORDER}.get(form, mfc.MFC_RECON_WENO5)
    q0 = oracle.prim_to_cons_field(spec, w)
    q, t = run(spec, q0, 3, recon, precision)
    p, tp = run(spec, q0, 3, recon, precision, stages=True)
    # the same arithmetic in other kernels: a few roundings of each stage, amplified by the pressure recovery
    bar = 1e-10 if precision == mfc.MFC_FP64 else 1e-4
    assert (rel_linf(q, p, spec) <= bar).all() and abs(t[0] - tp[0]) <= bar * tp[0]


def test_many_pieces():
    n = 130000
    spec, w = W.shock_tube_1d(n)
    q0 = oracle.prim_to_cons_field(spec, w)
    q, t = run(spec, q0, 3)
    p, tp = run(spec, q0, 3, stages=True)
    assert (rel_linf(q, p, spec) <= 1e-10).all() and abs(t[0] - tp[0]) <= 1e-10 * tp[0]
