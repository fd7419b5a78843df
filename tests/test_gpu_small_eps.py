"""Uniform and partly uniform grids with an epsilon whose eighth power (WENO5)
or fourth power (WENO3) FP64 can't hold, through every kernel, against the
oracle."""
import dataclasses
import sys

import pytest

import oracle
from parity_util import rel_linf, rhs_err, rounding_spread, step_bar
from paper_2305_09163_amd import mfc
from paper_2305_09163_amd import workloads as W

pytestmark = pytest.mark.gpu

RECON = {5: (mfc.MFC_RECON_WENO5, oracle.RECON_WENO5), 3: (mfc.MFC_RECON_WENO3, oracle.RECON_WENO3)}
CASES = {"tube": (lambda: W.shock_tube_1d(200), (0, 1)), "droplet": (lambda: W.droplet_shock_2d((40, 33), W.SEED + 11), (0, 1)),
         "bubble": (lambda: W.bubble_collapse_3d(n=(17, 15, 17)), (0, 1, 2)),
         "bubble stretched in x": (lambda: W.bubble_collapse_3d(n=(17, 15, 17)), (0, 2))}


@pytest.mark.parametrize("eps", [1e-40, 1e-120])
@pytest.mark.parametrize("name,kernel,order", [(n, k, o) for n, (_, ks) in CASES.items() for k in ks for o in (5, 3)
                                               if o == 5 or "stretched" not in n])
def test_rhs_and_step(name, kernel, order, eps):
    print(f"[small eps] {name} kernel {kernel} order {order} eps {eps:g}", file=sys.stderr, flush=True)
    spec, w = CASES[name][0]()
    spec = dataclasses.replace(spec, weno_eps=eps)
    if "stretched" in name:
        spec = dataclasses.replace(spec, faces=(W.tanh_faces(17, depth=0.6), None, None))
    rg, ro = RECON[order]
    q0 = oracle.prim_to_cons_field(spec, w)
    s = mfc.Solver(spec, kernel=kernel, recon=rg)
    q = s.upload(q0)
    s.fill_ghosts(q)
    r = s.rhs(q).cpu().numpy()
    s.check()
    qo = oracle.fill_ghosts(spec, q0)
    ref, st = oracle.rhs(spec, qo, recon=ro)
    assert st == oracle.OK
    assert rhs_err(r, ref, qo, spec).max() <= 1e-12
    q = s.upload(q0)
    s.step(q, cfl=0.3)
    s.check()
    qn, _, st = oracle.run(spec, q0, 1, cfl=0.3, recon=ro)
    assert st == oracle.OK
    bar = step_bar(rounding_spread(spec, q0, 1, cfl=0.3, recon=ro))
    err = rel_linf(q.cpu().numpy(), qn, spec)
    assert (err <= bar).all(), (err, bar)
