"""Wave-speed workgroups of uneven batched runs: from one for the smallest run
to the most a run takes, beside each other.  Single steps (which reduce the
wave speeds of their own input) give the step sizes and states of the runs
alone, bit for bit."""
import sys

import pytest
import torch

import oracle
from paper_2305_09163_amd import mfc
from paper_2305_09163_amd import workloads as W

pytestmark = pytest.mark.gpu

# 9 cells; 256 and 257 (one workgroup and two); 16384 and more (the most)
SIZES = [(3, 3), (16, 16), (257, 3), (128, 128), (131, 129), (5, 7)]


@pytest.mark.parametrize("precision", [mfc.MFC_FP64, mfc.MFC_FP32_MIXED])
def test_uneven_runs(precision):
    print(f"[batch small] precision {precision}", file=sys.stderr, flush=True)
    runs = [W.droplet_shock_2d(n, W.SEED + 40 + i) for i, n in enumerate(SIZES)]
    b = mfc.Batch([s for s, _ in runs], precision=precision)
    qi = [oracle.prim_to_cons_field(s, w) for s, w in runs]
    qs = b.upload(qi)
    for _ in range(3):
        b.step(qs, 0.3)
    b.check()
    times = b.time()
    for (spec, _), q, q0, t in zip(runs, qs, qi, times):
        s = mfc.Solver(spec, precision=precision)
        d = s.upload(q0)
        for _ in range(3):
            s.step(d, cfl=0.3)
        s.check()
        assert s.time()[0] == t and torch.equal(q[spec.interior], d[spec.interior]), spec.n
