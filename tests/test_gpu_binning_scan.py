"""The scan of the binning: one or two kernels after the per-block sums (up to 1024 blocks of 4096
anchors each block adds up its predecessors itself), lists of work items by 1024 or 4096 anchors
a workgroup, and passes with and without a list of short items (16 samples per anchor).

Every sample must stand exactly once in the anchor order, and the time-ordered data must equal
that of a batch, whose gather takes all items in one list, bit for bit.
"""
import numpy as np
import pytest
import torch

import workloads as W
from paper_2201_03478_amd import api

pytestmark = pytest.mark.gpu


# anchors: 32 -> 9 000, 300 -> 0.8e6, 360 -> 1.2e6 (4096 a workgroup), 660 -> 3.6e6 and 720 ->
# 4.25e6 (three kernels)
@pytest.mark.parametrize("L,n", [(32, 4097), (32, 100_000), (32, 157_000), (32, 158_000), (32, 400_000), (300, 50_000), (360, 50_000), (660, 30_000),
                                 (720, 30_000)])
def test_every_sample_once(L, n):
    K = 2
    a, b = (torch.from_numpy(v).cuda() for v in (W.sky_alm(L, 61), W.beam_alm(L, K, 62, kind="flat")))
    p_np = W.uniform_pointings(n, 63)
    p_np[0, 0], p_np[1, 0] = 0.0, np.pi
    p = torch.from_numpy(p_np).cuda()
    plan = api.Plan(L, K)
    got = plan.convolve(a, b, p)
    order = plan.debug_stage(2, n).cpu().numpy()
    assert np.array_equal(np.sort(order), np.arange(n, dtype=np.int32))
    (ref,) = api.Batch([dict(lmax=L, kmax=K, blm=b, ptg=p)], L).run(a, use_graph=False)
    torch.cuda.synchronize()
    assert torch.equal(got, ref)
