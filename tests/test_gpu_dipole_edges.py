"""Dipole response at the edges of a workgroup's 512 samples and of its velocity periods.

The reference is the same call on one sample at a time with the sample's own velocity: the
same operations, so the results agree bit for bit.
"""
import numpy as np
import pytest
import torch

import workloads as W
from paper_2201_03478_amd import api

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 511, 512, 513, 1025])
@pytest.mark.parametrize("spp", [1, 2, 255, 511, 512, 513, 1024])
def test_dipole_edges(n, spp):
    b = torch.from_numpy(W.beam_alm(4, 2, 71)).cuda()
    base = torch.from_numpy(W.uniform_pointings(n + 1, 72)).cuda()
    ptg = base[1:]  # 24 bytes in: the loads are 8-byte aligned only
    beta = torch.from_numpy(np.random.default_rng(73).standard_normal((-(-n // spp), 3)) * 1e-4).cuda()
    got = api.dipole_response(b, 4, 2, ptg, beta, spp, 2.7255, 1.3)
    per = beta[torch.arange(n, device="cuda") // spp].contiguous()
    for i in sorted({0, 1, spp - 1, spp, spp + 1, 510, 511, 512, 513, n - 2, n - 1}):
        if 0 <= i < n:
            one = api.dipole_response(b, 4, 2, ptg[i:i + 1].clone(), per[i:i + 1].clone(), 1, 2.7255, 1.3)
            assert torch.equal(got[i:i + 1], one), i
