"""Installing a network waits for its own upload, not for the device: work on
another stream goes on beside it."""
import sys

import numpy as np
import pytest
import torch

from oracle import indicator as ind
from paper_2305_09163_amd import mfc
from paper_2305_09163_amd import workloads as W

pytestmark = pytest.mark.gpu


def test_does_not_wait_for_other_streams():
    print("[set_indicator] beside another stream's work", file=sys.stderr, flush=True)
    params = ind.flatten(ind.init_params(5)).astype(np.float32)
    s = mfc.Solver(W.bubble_collapse_3d(n=8)[0], recon=mfc.MFC_RECON_LEARNED)
    s.set_indicator(params, 0.5)   # allocates, loads the kernel
    a = torch.ones((8192, 8192), device="cuda")
    b = torch.empty_like(a)
    side, done = torch.cuda.Stream(), torch.cuda.Event()
    torch.mm(a, a, out=b)
    torch.cuda.synchronize()
    with torch.cuda.stream(side):   # of the order of a second
        for _ in range(80):
            torch.mm(a, a, out=b)
        done.record()
    s.set_indicator(params, 0.25)
    running = not done.query()
    torch.cuda.synchronize()
    assert running
