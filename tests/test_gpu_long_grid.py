"""A 3D grid with more planes than four per workgroup fit into a launch's z
extent (65535): a state that repeats along z gives the right-hand side of one
period, bit for bit, and so does a step."""
import dataclasses
import sys

import pytest
import torch

import oracle
from paper_2305_09163_amd import mfc
from paper_2305_09163_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nz", [65560, 262200])
def test_long_grid_repeats_a_period(nz):
    print(f"[long grid] {nz}", file=sys.stderr, flush=True)
    period = 20

    def spec(n):
        s, w = W.bubble_collapse_3d(n=(4, 3, period))
        return dataclasses.replace(s, n=(4, 3, n), lo=(0.0, 0.0, 0.0), hi=(4.0, 3.0, float(n)), bc=(1,) * 6), w

    short, w = spec(period)
    long = spec(nz)[0]
    q0 = oracle.prim_to_cons_field(short, w)
    a, b = mfc.Solver(short, kernel=mfc.MFC_KERNEL_SPLIT), mfc.Solver(long, kernel=mfc.MFC_KERNEL_SPLIT)
    mfc.mfc_set_kernel_timing(a.h, True)   # the split kernels for the steps of the short grid as well
    qa = a.upload(q0)
    qb = b.empty()
    inner = slice(3, 3 + period)
    qb.zero_()
    qb[:, 3:-3] = qa[:, inner].repeat(1, nz // period, 1, 1)
    for step in (False, True):
        if step:
            a.step(qa, dt=1e-4)
            b.step(qb, dt=1e-4)
            ra, rb = qa, qb
        else:
            ra, rb = a.rhs(qa), b.rhs(qb)
        a.check()
        b.check()
        one = ra[short.interior]
        got = rb[long.interior].view(one.shape[0], nz // period, period, 3, 4)
        assert torch.equal(got, one[:, None].expand_as(got))
