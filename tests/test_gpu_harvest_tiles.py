"""Harvested samples on either side of the rule that gives every direction its
own workgroups (few tiles) or none: features, deviations and labels against
the oracle, with the smallest grid and ragged tiles."""
import sys

import numpy as np
import pytest
import torch

import oracle
from oracle import indicator as ind
from paper_2305_09163_amd import mfc
from paper_2305_09163_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [(3, 3, 3), (17, 9, 5), (24, 24, 24), (41, 33, 22), (3, 3), (70, 51), (300, 290)])
def test_tiles(n):
    print(f"[harvest tiles] {n}", file=sys.stderr, flush=True)
    spec = W.GridSpec(ndim=len(n), n=n, pi_inf=(0.0, 0.0), gamma=(1.5, 1.5))
    rng = np.random.default_rng(9)
    shape = spec.shape[1:]
    # random values exact in binary, so that both sides recover the same bits:
    # density one, pressure E / 2 (no kinetic energy), any volume fraction
    q = np.zeros(spec.shape)
    q[0] = rng.integers(0, 513, size=shape) / 1024.0
    q[1] = 1.0 - q[0]
    q[-2] = rng.integers(1024, 4096, size=shape) / 2.0
    q[-1] = rng.integers(1, 1024, size=shape) / 1024.0
    xo, yo, do = ind.harvest(spec, oracle.fill_ghosts(spec, q))
    x, y, d = mfc.Solver(spec).harvest(torch.tensor(q).cuda())
    bits = x.cpu().numpy().astype(np.uint16).astype(np.uint32) << 16
    f = bits.view(np.float32).astype(np.float64)
    np.testing.assert_array_equal(f[:, :15], ind.bf16(xo)[:, :15])
    assert (f[:, 15] == 0).all()
    # random stencils: a few dozen roundings of weights up to one
    assert np.abs(d.cpu().numpy() - do).max() <= 1e-9
    clear = np.abs(do - 0.01) > 1e-6
    assert (y.cpu().numpy()[clear] == yo[clear]).all()
