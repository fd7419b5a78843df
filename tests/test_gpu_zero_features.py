"""Wavefronts whose indicator inputs are all zero skip the network: a state of
uniform alpha1, rho and p (exact in binary, so that every recovered pressure
has the same bits) with a varying velocity has only such stencils.  A network
that calls them smooth must give the all-linear right-hand side, one that does
not the all-WENO5 one, bit for bit; with one cell's pressure raised, the
wavefronts around it take the network itself and agree."""
import sys

import numpy as np
import pytest
import torch

from oracle import indicator as ind
from paper_2305_09163_amd import mfc
from paper_2305_09163_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,kernel", [((20, 18, 16), mfc.MFC_KERNEL_SPLIT), ((20, 18, 16), mfc.MFC_KERNEL_FUSED),
                                      ((40, 33), mfc.MFC_KERNEL_FUSED), ((300,), mfc.MFC_KERNEL_FUSED)])
@pytest.mark.parametrize("precision", [mfc.MFC_FP64, mfc.MFC_FP32_MIXED])
@pytest.mark.parametrize("bump", [False, True])
def test_zero_features(n, kernel, precision, bump):
    print(f"[zero features] {n} kernel {kernel} precision {precision} bump {bump}", file=sys.stderr, flush=True)
    nd = len(n)
    spec = W.GridSpec(ndim=nd, n=n, weno_eps=1e-6)
    rng = np.random.default_rng(4)
    shape = tuple(x + 6 for x in reversed(n))
    q = np.zeros((4 + nd,) + (1,) * (3 - nd) + shape)
    q[0], q[1], q[-1] = 2.0 ** -10, 1.0 - 2.0 ** -10, 2.0 ** -20
    u = rng.integers(-32, 33, size=(nd,) + q.shape[1:]) / 8.0
    q[2:2 + nd] = u
    q[-2] = 2.0 ** 19 + 0.5 * (u ** 2).sum(0)
    if bump:
        q[(-2,) + tuple(s // 2 for s in q.shape[1:])] += 4096.0

    def rhs(sign, tau):
        p = ind.init_params(5)
        p["W3"] = p["W3"] * 0.0
        p["b3"] = p["b3"] * 0.0 + sign * 8.0
        s = mfc.Solver(spec, precision=precision, recon=mfc.MFC_RECON_LEARNED, kernel=kernel)
        s.set_indicator(ind.flatten(p).astype(np.float32), tau)
        d = s.upload(q)
        s.fill_ghosts(d)
        r = s.rhs(d)
        s.check()
        return r

    linear, weno = rhs(1.0, 0.0), rhs(1.0, 1.0)
    assert not torch.equal(linear, weno)
    assert torch.equal(rhs(1.0, 0.5), linear)
    assert torch.equal(rhs(-1.0, 0.5), weno)
