"""A batch in which some runs have characteristic faces: the others still give
the bits of the same run advanced alone."""
import dataclasses
import sys

import pytest
import torch

import oracle
from paper_2305_09163_amd import mfc
from paper_2305_09163_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [mfc.MFC_FP64, mfc.MFC_FP32_MIXED])
def test_runs_beside_characteristic_ones_keep_their_bits(precision):
    print(f"[batch mixed] precision {precision}", file=sys.stderr, flush=True)
    runs = []
    for i, (n, bc) in enumerate([((33, 27), (2, 0, 0, 2, 0, 0)), ((40, 17), (0,) * 6), ((19, 23), (1, 1, 1, 1, 0, 0)),
                                 ((64, 35), (1, 1, 0, 0, 0, 0))]):
        spec, w = W.droplet_shock_2d(n, W.SEED + 700 + i)
        runs.append((dataclasses.replace(spec, bc=bc), w))
    b = mfc.Batch([s for s, _ in runs], precision=precision)
    qi = [oracle.prim_to_cons_field(s, w) for s, w in runs]
    for shape in range(3):
        b.set_tune(shape, 1, 1)
        qs = b.upload(qi)
        b.run(qs, 5, 0.3, use_graph=False)
        b.check()
        for (spec, _), q, q0 in zip(runs[1:], qs[1:], qi[1:]):
            s = mfc.Solver(spec, precision=precision)
            d = s.upload(q0)
            s.run(d, 5, cfl=0.3)
            s.check()
            assert torch.equal(q[spec.interior], d[spec.interior]), (shape, spec.n)
