"""bin_chunk: an upper limit of the samples per work item, on which results do not depend."""
import numpy as np
import pytest
import torch

import workloads as W
from paper_2201_03478_amd import api, autotune

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "f64maps_f32gather", "mixed"])
@pytest.mark.parametrize("n", [4000, 30_000])
def test_data_do_not_depend_on_it(prec, n):
    """Items of 1 to n samples: a third of the pointings in one cell, a third in forty."""
    L, K = 24, 5
    a, b = (torch.from_numpy(v).cuda() for v in (W.sky_alm(L, 5), W.beam_alm(L, K, 6, kind="flat")))
    p_np = W.uniform_pointings(n, 7)
    p_np[:n // 3, :2] = 1.0 + 1e-3 * p_np[:n // 3, :2] / 7
    p_np[n // 3:2 * n // 3, :2] = 0.5 + 0.5 * p_np[n // 3:2 * n // 3, :2] / 7
    p = torch.from_numpy(np.ascontiguousarray(p_np)).cuda()
    plan = api.Plan(L, K, prec)
    ref = plan.convolve(a, b, p).clone()
    for c in (16, 17, 64, 100, 128, 256, 1000, 1 << 20):
        plan.set_param("bin_chunk", c)
        assert plan.get_param("bin_chunk") == c
        assert torch.equal(plan.convolve(a, b, p), ref), c


def test_tuner_tries_no_chunk_twice():
    """FP64 work items hold at most 128 samples, so the tuner has no larger chunks to try there."""
    assert len([c for c in autotune.BIN_CHUNK[api.N.SC_FP64] if c > 128]) == 1
