"""Short work items of the split FP32-map gather, and the one-workgroup binning of small passes.

A plan's gather sends items of at most 16 samples to a wave-per-item kernel, and bins passes
of at most 4096 samples in one workgroup; a batch always takes the workgroup gather.  Both
form the same products in the same order, so the two agree bit for bit.
"""
import numpy as np
import pytest
import torch

import workloads as W
from paper_2201_03478_amd import api

pytestmark = pytest.mark.gpu


def _clusters(info, n, seed):
    """n pointings in cells of 1 to 40 samples, in random order, the poles among them."""
    rng = np.random.default_rng(seed)
    hth, hph = 2 * np.pi / info["n_theta_fine"], 2 * np.pi / info["n_phi"]
    cell = np.repeat(np.arange(n), 1 + np.arange(n) % 40)[:n]
    r = rng.integers(0, info["n_theta_fine"] // 2, n)[cell]
    c = rng.integers(0, info["n_phi"], n)[cell]
    p = np.stack([(r + rng.uniform(0.01, 0.99, n)) * hth, (c + rng.uniform(0.01, 0.99, n)) * hph,
                  rng.uniform(0, 2 * np.pi, n)], 1)
    p[0], p[-1] = [0.0, 1.0, 0.3], [np.pi, 2.0, 0.4]
    return torch.from_numpy(np.ascontiguousarray(p[rng.permutation(n)])).cuda()


@pytest.mark.parametrize("kmax", [0, 7, 8, 40, 71, 72, 100])
@pytest.mark.parametrize("n", [1, 2, 63, 1024, 1025, 4095, 4096, 4097, 20_000])
def test_short_items_equal_the_workgroup_gather(kmax, n):
    L = max(kmax, 40)
    a = torch.from_numpy(W.sky_alm(L, 61)).cuda()
    b = torch.from_numpy(W.beam_alm(L, kmax, 62, kind="flat")).cuda()
    plan = api.Plan(L, kmax)
    ptg = _clusters(plan.info(), n, 63 + n)
    got = plan.convolve(a, b, ptg)
    order = plan.debug_stage(2, n).cpu().numpy()
    assert np.array_equal(np.sort(order), np.arange(n, dtype=np.int32))
    (ref,) = api.Batch([dict(lmax=L, kmax=kmax, blm=b, ptg=ptg)], L).run(a, use_graph=False)
    torch.cuda.synchronize()
    assert torch.equal(got, ref)
