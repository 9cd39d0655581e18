"""Ring-sum layouts with more than four rings per lane (the plan's own choice when enough
(m, k) columns remain).

A ring's sums do not depend on which lane forms them, so the plan's choice must give the
time-ordered data of every layout set through ring_rpt bit for bit.  The band limits take
5, 7, 8 and 9 rings per lane, the first and last of a layout among them, and steps that
end within an iteration of four.
"""
import numpy as np
import pytest
import torch

import workloads as W
from paper_2201_03478_amd import api

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "f64maps_f32gather"])
@pytest.mark.parametrize("L,K", [(270, 17), (310, 15), (384, 12), (415, 11), (440, 10), (487, 9), (512, 8), (513, 9)])
def test_layouts_agree(prec, L, K):
    a, b = (torch.from_numpy(v).cuda() for v in (W.sky_alm(L, 5), W.beam_alm(L, K, 6, kind="flat")))
    p_np = W.uniform_pointings(500, 7)
    p_np[0, 0], p_np[1, 0] = 0.0, np.pi
    p = torch.from_numpy(p_np).cuda()
    plan = api.Plan(L, K, prec)
    own = plan.get_param("ring_rpt")
    ref = plan.convolve(a, b, p).clone()
    for r in (1, 2, 3, 4):
        if r == own:
            continue
        plan.set_param("ring_rpt", r)
        assert plan.get_param("ring_rpt") == r
        assert torch.equal(plan.convolve(a, b, p), ref), "ring_rpt %d" % r
    plan.set_param("ring_rpt", own)
    assert torch.equal(plan.convolve(a, b, p), ref)
