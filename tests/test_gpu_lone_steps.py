"""Single steps on either side of the largest non-uniform 1D grids that take
them in one launch, against the oracle."""
import dataclasses
import sys

import pytest

import oracle
from parity_util import acoustic_floor, rel_l1, rel_linf, rounding_spread, step_bar
from paper_2305_09163_amd import mfc
from paper_2305_09163_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,n", [(mfc.MFC_FP64, 574), (mfc.MFC_FP64, 575), (mfc.MFC_FP64, 1022),
                                         (mfc.MFC_FP32_MIXED, 638), (mfc.MFC_FP32_MIXED, 639)])
@pytest.mark.parametrize("bc", [0, 1])
def test_stretched_step(precision, n, bc):
    print(f"[lone step] {n} precision {precision} bc {bc}", file=sys.stderr, flush=True)
    spec, w = W.shock_tube_1d(n)
    spec = dataclasses.replace(spec, bc=(bc,) * 6, faces=(W.tanh_faces(n, centre=0.7, depth=0.5), None, None))
    q0 = oracle.prim_to_cons_field(spec, w)
    s = mfc.Solver(spec, precision=precision)
    q = s.upload(q0)
    s.step(q, cfl=0.3)
    s.check()
    qn, t, st = oracle.run(spec, q0, 1, cfl=0.3)
    assert st == oracle.OK
    got = q.double().cpu().numpy()
    if precision == mfc.MFC_FP64:
        bar = step_bar(rounding_spread(spec, q0, 1, cfl=0.3))
        err = rel_linf(got, qn, spec)
        assert abs(s.time()[0] - t) <= 1e-12 * t
    else:   # the bar of FP32 runs
        bar = 1e-4
        err = rel_l1(got, qn, spec, floor_mom=acoustic_floor(spec, q0))
    assert (err <= bar).all(), (err, bar)
