"""Work items of at most 16 samples of the FP64 gather: every count, every remainder of the
component quads, every kernel width.

The reference is the per-sample path (SC_GATHER_PATH=direct): the same interpolation with
FP64 sums in another order, a few hundred additions of relative error 2^-53 each, so 1e-12 of
the largest value bounds the difference.
"""
import os

import numpy as np
import pytest
import torch

import workloads as W
from paper_2201_03478_amd import api

pytestmark = pytest.mark.gpu


def _plan(direct, *args, **kw):
    old = os.environ.pop("SC_GATHER_PATH", None)
    try:
        if direct:
            os.environ["SC_GATHER_PATH"] = "direct"
        return api.Plan(*args, **kw)
    finally:
        os.environ.pop("SC_GATHER_PATH", None)
        if old is not None:
            os.environ["SC_GATHER_PATH"] = old


@pytest.mark.parametrize("width", [4, 6, 8, 10, 12, 14, 16])
@pytest.mark.parametrize("kmax", [0, 1, 2, 3, 4, 5, 6, 7, 9, 20])
def test_short_fp64_items(width, kmax):
    L = 24
    a = torch.from_numpy(W.sky_alm(L, 91)).cuda()
    b = torch.from_numpy(W.beam_alm(L, kmax, 92, kind="flat")).cuda()
    plan, ref = (_plan(d, L, kmax, "fp64", kernel_width=width) for d in (False, True))
    info = plan.info()
    rng = np.random.default_rng(93)
    hth, hph = 2 * np.pi / info["n_theta_fine"], 2 * np.pi / info["n_phi"]
    p = [np.stack([((5 * c) % (info["n_theta_fine"] // 2) + rng.uniform(0.01, 0.99, c)) * hth,
                   ((7 * c) % info["n_phi"] + rng.uniform(0.01, 0.99, c)) * hph, rng.uniform(0, 2 * np.pi, c)], 1)
         for c in range(1, 18)]
    p.append(np.array([[0.0, 1.0, 0.3], [np.pi, 2.0, 0.4], [1.0, 2 * np.pi - 1e-9, 0.5]]))
    p = np.concatenate(p)
    ptg = torch.from_numpy(np.ascontiguousarray(p[rng.permutation(len(p))])).cuda()
    want = ref.convolve(a, b, ptg)
    for reps in (1, 30):  # one workgroup's binning; the general one, with longer items beside
        q = torch.cat([ptg] + [ptg[:173]] * (reps - 1))
        got = plan.convolve(a, b, q)[:len(p)]
        assert float((got - want).abs().max()) <= 1e-12 * float(want.abs().max())
