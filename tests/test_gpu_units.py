"""States in units that make density and pressure very small or very large:
with densities and pressures multiplied by the same power of two, velocities,
sound speeds and volume fractions stay, so every conserved row of a
first-order right-hand side takes that factor and the volume fraction's
none.  The products the flux forms of both (density times pressure) leave the
type's range although each factor is well within it."""
import dataclasses
import sys

import numpy as np
import pytest
import torch

import oracle
from paper_2305_09163_amd import mfc
from paper_2305_09163_amd import workloads as W

pytestmark = pytest.mark.gpu

GRIDS = {"1d": (lambda: W.shock_tube_1d(200), mfc.MFC_KERNEL_FUSED),
         "2d": (lambda: W.droplet_shock_2d((40, 33), W.SEED + 11), mfc.MFC_KERNEL_FUSED),
         "3d split": (lambda: W.bubble_collapse_3d(n=(17, 15, 17)), mfc.MFC_KERNEL_SPLIT)}


@pytest.mark.parametrize("grid", sorted(GRIDS))
@pytest.mark.parametrize("precision,k", [(mfc.MFC_FP64, -600), (mfc.MFC_FP64, 560), (mfc.MFC_FP32_MIXED, -84),
                                         (mfc.MFC_FP32_MIXED, 70)])
def test_scaled_density_and_pressure(grid, precision, k):
    print(f"[units] {grid} precision {precision} 2^{k}", file=sys.stderr, flush=True)
    make, kernel = GRIDS[grid]
    spec, w = make()
    nd = spec.ndim
    # gases (no stiffness), pressures of order 1, the workload's own densities scaled to order 1
    spec = dataclasses.replace(spec, pi_inf=(0.0, 0.0))
    w = w.copy()
    w[0] /= 1000.0
    w[1] /= 1000.0
    w[2 + nd] = 1.0 + (w[2 + nd] > w[2 + nd].mean())
    w[2] = 0.25
    q = oracle.prim_to_cons_field(spec, w)
    scale = np.ones((spec.nvar, 1, 1, 1))
    scale[:-1] = 2.0 ** k
    out = []
    for f in (np.ones_like(scale), scale):
        s = mfc.Solver(spec, precision=precision, recon=mfc.MFC_RECON_FIRST_ORDER, kernel=kernel)
        d = s.upload(q * f)
        s.fill_ghosts(d)
        r = s.rhs(d)
        s.step(d, cfl=0.3)
        s.check()
        out.append((r[spec.interior].double().cpu().numpy() / f, d[spec.interior].double().cpu().numpy() / f))
    # the sound speed may be rounded another way: a few units in the last place
    # of fluxes and their sums, against the largest value
    tol = 64 * (np.finfo(np.float64).eps if precision == mfc.MFC_FP64 else np.finfo(np.float32).eps)
    for a, b in zip(*out):
        flat = lambda x: np.abs(x).reshape(spec.nvar, -1).max(axis=1)
        assert (flat(a - b) <= tol * max(flat(a).max(), 1.0)).all(), flat(a - b)
