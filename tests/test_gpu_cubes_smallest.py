"""One-launch stages on the smallest 3D grids, periodic: a stencil past one
face wraps onto the cells past the other.  Three steps against the split
kernels (taken while kernel timing is on), the ghost cells left alone, and
single steps with the step sizes they report."""
import dataclasses
import sys

import pytest
import torch

import oracle
from parity_util import rel_linf
from paper_2305_09163_amd import mfc
from paper_2305_09163_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [(3, 3, 3), (4, 3, 5), (3, 10, 3), (16, 4, 3)])
@pytest.mark.parametrize("bc", [(1,) * 6, (1, 1, 0, 0, 1, 1)])
def test_smallest_periodic(n, bc):
    spec, w = W.bubble_collapse_3d(n=n)
    spec = dataclasses.replace(spec, bc=bc)
    print(f"[cubes smallest] {n} bc {bc}", file=sys.stderr, flush=True)
    q0 = oracle.prim_to_cons_field(spec, w)
    out = []
    for split in (False, True):
        s = mfc.Solver(spec, kernel=mfc.MFC_KERNEL_SPLIT)
        if split:
            mfc.mfc_set_kernel_timing(s.h, True)
        q = s.upload(q0)
        s.run(q, 3, cfl=0.3)
        s.check()
        out.append((q, s.time()))
    (q, t), (p, tp) = out
    # The two round each stage once or twice differently, in water a stage's
    # rounding moves a momentum at rest by about 2e-12 of the largest (the
    # pressure recovery subtracts Pi): six roundings over three steps.
    bar = 1.2e-11
    err = rel_linf(q.cpu().numpy(), p.cpu().numpy(), spec)
    assert (err <= bar).all(), err
    assert abs(t[0] - tp[0]) <= bar * tp[0]
    ghosts = torch.ones(q.shape[1:], dtype=torch.bool, device="cuda")
    ghosts[spec.interior[1:]] = False
    assert torch.equal(q[:, ghosts], s.upload(q0)[:, ghosts])
    s = mfc.Solver(spec, kernel=mfc.MFC_KERNEL_SPLIT)
    one, dt, total = s.upload(q0), torch.zeros((), dtype=torch.float64, device="cuda"), 0.0
    for _ in range(3):
        s.step(one, cfl=0.3, dt_used=dt)
        total += dt.item()
    s.check()
    assert s.time() == (total, dt.item())
    assert (rel_linf(one.cpu().numpy(), p.cpu().numpy(), spec) <= bar).all()
