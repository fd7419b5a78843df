"""The gradient reduction at the edges of its rows (64 workgroup partials are
added per pass): a batch of 2^k copies of one sample has that sample's
gradient, whatever the number of partials, with idle workgroups among them.
Scaling by 2^-k is exact in FP32 and bf16, so only the order of the sums
differs: at most one rounding per addend."""
import sys

import numpy as np
import pytest
import torch

from oracle import indicator as ind
from paper_2305_09163_amd import mfc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("max_batch,batch", [(16, 16), (4096, 4096), (4160, 4096), (8192, 8192), (8256, 8192),
                                             (65536, 65536)])
def test_copies_of_one_sample(max_batch, batch):
    print(f"[reduce] {batch} of {max_batch}", file=sys.stderr, flush=True)
    rng = np.random.default_rng(3)
    w = ind.flatten(ind.init_params(5)).astype(np.float32)
    x = (rng.normal(size=(1, 16)).astype(np.float32).view(np.uint32) >> 16).astype(np.uint16).view(np.int16)
    x[0, 15] = 0
    X, Y = torch.tensor(x).cuda(), torch.ones(1, dtype=torch.uint8, device="cuda")
    one = mfc.Trainer(1)
    one.set_params(w)
    one.grad(X, Y)
    g1, l1 = one.read_grad()
    t = mfc.Trainer(max_batch)
    t.set_params(w)
    t.grad(X, Y, torch.zeros(batch, dtype=torch.int32, device="cuda"))
    g, loss = t.read_grad()
    bar = (batch / 64 + 16 + 4 + 512) * 2.0 ** -23   # addends per chain: tiles of a wavefront, samples, wavefronts, workgroups
    assert np.abs(g - g1).max() <= bar * np.abs(g1).max() and (np.abs(g - g1) <= bar * np.abs(g1) + 1e-30).all()
    assert abs(loss - l1) <= bar * abs(l1)
