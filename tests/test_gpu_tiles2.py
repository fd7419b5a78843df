"""The 2D tile kernels at the edges of their 16 x 14 tiles, alone and batched:
grids below one tile, exactly one, one cell over, and one of more tiles than a
first stage reduces wave speeds for itself.  A run of three steps (whose later
steps take the speeds the stage before left) against the oracle, the ghost
cells it leaves, and the bare right-hand side on the caller's own ghost cells."""
import dataclasses
import sys

import numpy as np
import pytest
import torch

import oracle
from parity_util import rel_linf, rhs_err, rounding_spread_run, step_bar
from paper_2305_09163_amd import mfc
from paper_2305_09163_amd import workloads as W

pytestmark = pytest.mark.gpu

GRIDS = [(3, 3), (16, 14), (17, 15), (15, 29), (50, 43), (370, 330)]


@pytest.mark.parametrize("n", GRIDS)
@pytest.mark.parametrize("bc", [0, 1, 2])
def test_tiles(n, bc):
    spec, w = W.droplet_shock_2d(n, W.SEED + 31)
    spec = dataclasses.replace(spec, bc=(bc,) * 6)
    print(f"[tiles2] {n} bc {bc}", file=sys.stderr, flush=True)
    q0 = oracle.prim_to_cons_field(spec, w)
    s = mfc.Solver(spec)
    qf = oracle.fill_ghosts(spec, q0)
    r = s.rhs(s.upload(qf)).cpu().numpy()
    ref, st = oracle.rhs(spec, qf)
    assert st == oracle.OK
    assert rhs_err(r, ref, qf, spec).max() <= 1e-12
    q, half = s.upload(q0), s.upload(q0)
    s.run(q, 3, cfl=0.3)
    s.check()
    qn, _, st = oracle.run(spec, q0, 3, cfl=0.3)
    assert st == oracle.OK
    # 1e-12 per variable, or twice the oracle's own rounding-order spread over the same run
    bar = step_bar(rounding_spread_run(spec, q0, 3, cfl=0.3, norm="linf"))
    err = rel_linf(q.cpu().numpy(), qn, spec)
    assert (err <= bar).all(), (err, bar)
    # single steps take the same path, and the run's ghost cells are those of its last step's start
    s.run(half, 2, cfl=0.3)
    s.fill_ghosts(half)
    inner = (slice(None),) + spec.interior[1:]
    ghosts = torch.ones(q.shape[1:], dtype=torch.bool, device="cuda")
    ghosts[spec.interior[1:]] = False
    assert torch.equal(q[:, ghosts], half[:, ghosts])
    s.step(half, cfl=0.3)
    assert torch.equal(q[inner], half[inner])
    # the batch takes the same tiles
    if bc != 2:
        b = mfc.Batch([spec, spec], precision=mfc.MFC_FP64)
        qs = [s.upload(q0), s.upload(q0)]
        b.run(qs, 3, 0.3)
        b.check()
        for x in qs:
            assert torch.equal(x[inner], q[inner])


def test_rhs_reads_the_callers_ghost_cells():
    spec, w = W.droplet_shock_2d((33, 20), W.SEED + 32)
    q0 = oracle.fill_ghosts(spec, oracle.prim_to_cons_field(spec, w))
    q1 = q0.copy()
    q1[:, :, 3:-3, :3] *= 1.01   # an inflow of the caller's own on the low x face
    s = mfc.Solver(spec)
    r = s.rhs(s.upload(q1)).cpu().numpy()
    ref, st = oracle.rhs(spec, q1)
    assert st == oracle.OK
    assert rhs_err(r, ref, q1, spec).max() <= 1e-12
    assert not np.array_equal(ref, oracle.rhs(spec, q0)[0])
