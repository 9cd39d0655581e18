"""ring_rpt: the plan's own layout is read back, every layout can be set, and no other value.

A ring's sums do not depend on the lane that forms them, so every layout gives the same bits.
"""
import pytest
import torch

import workloads as W
from paper_2201_03478_amd import api

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "f64maps_f32gather"])
@pytest.mark.parametrize("L,K,own", [(32, 1, 1), (64, 1, 2), (128, 1, 3), (700, 3, 4), (270, 17, 5), (310, 15, 5),
                                     (384, 12, 7), (415, 11, 7), (440, 10, 8), (487, 9, 8), (512, 8, 9), (513, 9, 9)])
def test_every_layout(prec, L, K, own):
    a, b = (torch.from_numpy(v).cuda() for v in (W.sky_alm(L, 5), W.beam_alm(L, K, 6, kind="flat")))
    p = torch.from_numpy(W.uniform_pointings(300, 7)).cuda()
    plan = api.Plan(L, K, prec)
    assert plan.get_param("ring_rpt") == own
    ref = plan.convolve(a, b, p).clone()
    for r in (1, 2, 3, 4, 5, 7, 8, 9, own):
        plan.set_param("ring_rpt", r)
        assert plan.get_param("ring_rpt") == r
        assert torch.equal(plan.convolve(a, b, p), ref), r
    for r in (-1, 0, 6, 10):
        with pytest.raises(api.N.ScError):
            plan.set_param("ring_rpt", r)
        assert plan.get_param("ring_rpt") == own


def test_mixed_layouts():
    plan = api.Plan(512, 8, "mixed")
    assert 1 <= plan.get_param("ring_rpt") <= 4
    for r in (0, 5, 9):
        with pytest.raises(api.N.ScError):
            plan.set_param("ring_rpt", r)
