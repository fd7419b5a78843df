"""Harvested deviations where the fourth powers of the smoothness indicators
leave FP64's range although the definition's squares do not: differences of
1e-46 with a weno_eps below them, and of 1e45."""
import dataclasses
import sys

import numpy as np
import pytest
import torch

import oracle
from oracle import indicator as ind
from paper_2305_09163_amd import mfc
from paper_2305_09163_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [(300,), (20, 33), (9, 10, 12)])
@pytest.mark.parametrize("kind", ["small", "large"])
def test_deviation(n, kind):
    print(f"[harvest range] {n} {kind}", file=sys.stderr, flush=True)
    nd = len(n)
    spec = W.GridSpec(ndim=nd, n=n, pi_inf=(0.0, 0.0), weno_eps=1e-150 if kind == "small" else 1e-6)
    rng = np.random.default_rng(8)
    q = np.zeros(spec.shape)
    q[0], q[1], q[-1] = 2.0 ** -10, 1.0 - 2.0 ** -10, 2.0 ** -20
    q[-2] = 2.0 ** 19
    if kind == "small":
        q[2] = 1e-46 * rng.random(spec.shape[1:])   # velocities; the pressure has equal bits everywhere
    else:
        q[0] = 1e45 * (1.0 + rng.random(spec.shape[1:]))
    _, yo, do = ind.harvest(spec, oracle.fill_ghosts(spec, q))
    s = mfc.Solver(spec)
    _, y, d = s.harvest(torch.tensor(q).cuda())
    y, d = y.cpu().numpy(), d.cpu().numpy()
    assert do.max() > 0.1   # the case has deviations to find
    # random stencils (no nearly equal indicators): a few dozen roundings of weights up to one
    assert np.abs(d - do).max() <= 1e-9
    clear = np.abs(do - 0.01) > 1e-6
    assert (y[clear] == yo[clear]).all()
