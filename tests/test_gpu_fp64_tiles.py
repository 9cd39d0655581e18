"""The FP64 matrix-core gather and scatter at the edges of their tiles.

Work items of 1 to 129 samples (one, two or four 16-sample tiles, the 64-sample items of
the gather, the 128-sample items of the scatter), component counts around the 16-wide
tiles, every kernel width.  The reference is the per-sample path (SC_GATHER_PATH=direct),
which evaluates the same interpolation with FP64 sums in another order: the two differ by
rounding only, at most a few hundred additions of relative error 2^-53 each, so 1e-12 of
the largest value bounds the difference.
"""
import os

import numpy as np
import pytest
import torch

import workloads as W
from paper_2201_03478_amd import api

pytestmark = pytest.mark.gpu

COUNTS = [1, 2, 15, 16, 17, 31, 32, 33, 47, 63, 64, 65, 127, 128, 129]


def _pointings(info, seed):
    """COUNTS[i] samples inside the i-th of a set of distinct anchor cells, shuffled; the poles too."""
    rng = np.random.default_rng(seed)
    hth, hph = 2 * np.pi / info["n_theta_fine"], 2 * np.pi / info["n_phi"]
    nr, nc = info["n_theta_fine"] // 2, info["n_phi"]
    rows = [(5 * i) % nr for i in range(len(COUNTS))]
    cols = [(7 * i) % nc for i in range(len(COUNTS) - 1)] + [nc - 1]
    p = [np.stack([(r + rng.uniform(0.01, 0.99, c)) * hth, (q + rng.uniform(0.01, 0.99, c)) * hph,
                   rng.uniform(0, 2 * np.pi, c)], 1) for c, r, q in zip(COUNTS, rows, cols)]
    p.append(np.array([[0.0, 1.0, 0.3], [np.pi, 2.0, 0.4]]))
    p = np.concatenate(p)
    return np.ascontiguousarray(p[rng.permutation(len(p))])


def _run(direct, L, K, width, a, b, seed):
    old = os.environ.pop("SC_GATHER_PATH", None)
    try:
        if direct:
            os.environ["SC_GATHER_PATH"] = "direct"
        plan = api.Plan(L, K, "fp64", kernel_width=width)
    finally:
        os.environ.pop("SC_GATHER_PATH", None)
        if old is not None:
            os.environ["SC_GATHER_PATH"] = old
    ptg = torch.from_numpy(_pointings(plan.info(), seed)).cuda()
    y = torch.from_numpy(np.random.default_rng(seed + 1).standard_normal(ptg.shape[0])).cuda()
    tod = plan.convolve(a, b, ptg)
    return tod.cpu().numpy(), plan.adjoint(b, ptg, y).cpu().numpy(), plan.adjoint_beam(a, ptg, y).cpu().numpy()


@pytest.mark.parametrize("width", [4, 6, 8, 10, 12, 14, 16])
@pytest.mark.parametrize("kmax", [0, 6, 7, 8, 15, 23])
def test_fp64_tiles_match_the_per_sample_path(width, kmax):
    L = 24
    a = torch.from_numpy(W.sky_alm(L, 41)).cuda()
    b = torch.from_numpy(W.beam_alm(L, kmax, 42, kind="flat")).cuda()
    got = _run(False, L, kmax, width, a, b, 43)
    ref = _run(True, L, kmax, width, a, b, 43)
    for g, r in zip(got, ref):
        assert np.max(np.abs(g - r)) <= 1e-12 * np.max(np.abs(r))
