"""Split kernels at the edges of their chunk rule: grids whose x-y planes end
within a z-pass workgroup of 256 columns (one column short, exactly full, two
columns over), chunks of one plane and a last chunk that is short, x+y
workgroups of one, two and four planes.  Right-hand side and a short run (whose
steps after the first take the wave speeds the z pass reduced) against the
oracle, with extrapolated and with characteristic faces."""
import dataclasses
import sys

import pytest

import oracle
from parity_util import rel_linf, rhs_err, rounding_spread_run, step_bar
from paper_2305_09163_amd import mfc
from paper_2305_09163_amd import workloads as W

pytestmark = pytest.mark.gpu

GRIDS = [(85, 3, 5), (16, 16, 7), (86, 3, 40), (33, 31, 37), (64, 48, 61), (90, 80, 76)]


@pytest.mark.parametrize("n", GRIDS)
@pytest.mark.parametrize("bc", [0, 2])
def test_chunks(n, bc):
    spec, w = W.bubble_collapse_3d(n=n)
    spec = dataclasses.replace(spec, bc=(bc,) * 6)
    print(f"[chunks] {n} bc {bc}", file=sys.stderr, flush=True)
    q0 = oracle.prim_to_cons_field(spec, w)
    s = mfc.Solver(spec, kernel=mfc.MFC_KERNEL_SPLIT)
    r = s.rhs(s.upload(q0)).cpu().numpy()
    s.check()
    qf = oracle.fill_ghosts(spec, q0)
    ref, st = oracle.rhs(spec, qf)
    assert st == oracle.OK
    assert rhs_err(r, ref, qf, spec).max() <= 1e-12
    q = s.upload(q0)
    s.run(q, 3, cfl=0.3)
    s.check()
    qn, _, st = oracle.run(spec, q0, 3, cfl=0.3)
    assert st == oracle.OK
    # 1e-12 per variable, or twice the oracle's own rounding-order spread over the same run
    bar = step_bar(rounding_spread_run(spec, q0, 3, cfl=0.3, norm="linf"))
    err = rel_linf(q.cpu().numpy(), qn, spec)
    assert (err <= bar).all(), (err, bar)
