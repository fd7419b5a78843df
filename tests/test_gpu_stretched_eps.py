"""Non-uniform WENO5 at the ends of FP64's range: a weno_eps whose eighth
power underflows (cells of exactly equal values have no other term), and
differences whose smoothness indicators' eighth powers overflow.  The
definition needs (eps + beta)^2 only, so such grids take the same bars as any
other."""
import dataclasses
import sys

import numpy as np
import pytest

import oracle
from parity_util import rel_linf, rhs_err, rounding_spread, step_bar
from paper_2305_09163_amd import mfc
from paper_2305_09163_amd import workloads as W

pytestmark = pytest.mark.gpu


def blast(n, scale):
    """Gases at rest, both pressures times `scale`, stretched cells."""
    spec, w = W.shock_tube_1d(n)
    spec = dataclasses.replace(spec, pi_inf=(0.0, 0.0), faces=(W.tanh_faces(n, centre=0.7, depth=0.5), None, None))
    w = w.copy()
    w[2], w[3] = 0.0, np.where(w[3] > w[3].mean(), 2.0, 1.0) * scale
    return spec, w


def stretched(sw, *faces):
    spec, w = sw
    return dataclasses.replace(spec, faces=tuple(faces) + (None,) * (3 - len(faces))), w


CASES = {
    # 1D: whole steps (and the bare right-hand side of the fused kernel)
    "tube_200": lambda: stretched(W.shock_tube_1d(200), W.tanh_faces(200, centre=0.7, depth=0.5)),
    "tube_700": lambda: stretched(W.shock_tube_1d(700), W.tanh_faces(700, centre=0.7, depth=0.5)),
    "droplet_40x33": lambda: stretched(W.droplet_shock_2d((40, 33), W.SEED + 11), W.tanh_faces(40, centre=0.4, depth=0.5),
                                       W.tanh_faces(33, depth=0.3)),
    "bubble_17x15x17": lambda: W.bubble_collapse_3d(n=(17, 15, 17), stretch=0.6),
}
KERNELS = {"fused": mfc.MFC_KERNEL_FUSED, "split": mfc.MFC_KERNEL_SPLIT}


def check(name, kernel, spec, w):
    print(f"[stretched eps {spec.weno_eps:g} {kernel}] {name}", file=sys.stderr, flush=True)
    q0 = oracle.prim_to_cons_field(spec, w)
    s = mfc.Solver(spec, kernel=KERNELS[kernel])
    q = s.upload(q0)
    s.fill_ghosts(q)
    r = s.rhs(q).cpu().numpy()
    s.check()
    qo = oracle.fill_ghosts(spec, q0)
    ro, st = oracle.rhs(spec, qo)
    assert st == oracle.OK
    assert rhs_err(r, ro, qo, spec).max() <= 1e-12
    q = s.upload(q0)
    s.run(q, 2, cfl=0.3)
    s.check()
    qn, _, st = oracle.run(spec, q0, 2, cfl=0.3)
    assert st == oracle.OK
    bar = step_bar(rounding_spread(spec, q0, 2, cfl=0.3))
    err = rel_linf(q.cpu().numpy(), qn, spec)
    assert (err <= bar).all(), (err, bar)


@pytest.mark.parametrize("eps", [1e-40, 1e-120])
@pytest.mark.parametrize("name,kernel", [(n, "fused") for n in sorted(CASES)] + [("bubble_17x15x17", "split")])
def test_small_eps(name, kernel, eps):
    spec, w = CASES[name]()
    check(name, kernel, dataclasses.replace(spec, weno_eps=eps), w)


def test_large_differences():
    check("blast_200", "fused", *blast(200, 1e30))
