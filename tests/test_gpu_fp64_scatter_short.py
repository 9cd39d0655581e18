"""The FP64 adjoint's binned scatter at the edges of its forms.

Anchors of 1 to 5 samples (up to four go to the wave form), around the 16-, 64- and 128-sample
edges of the matrix form, in passes binned by one workgroup (up to 4096 samples) and by the
general path, component counts around the 16- and 32-wide edges of both, every kernel width.
The passes are long enough that binning them pays (the stage times show that it ran).  The
reference is the per-sample path; the sums differ in order only: at most a few hundred
additions of relative error 2^-53 each, so 1e-12 of the largest value bounds the difference.
"""
import numpy as np
import pytest
import torch

import workloads as W
from paper_2201_03478_amd import api

pytestmark = pytest.mark.gpu

COUNTS = [1, 2, 3, 4, 5, 1, 2, 3, 4, 15, 16, 17, 1, 31, 33, 63, 64, 65, 4, 127, 128, 129]


def _pointings(info, n, seed):
    """n pointings, COUNTS[i] in the i-th of a set of distinct anchor cells, shuffled; both poles."""
    rng = np.random.default_rng(seed)
    hth, hph = 2 * np.pi / info["n_theta_fine"], 2 * np.pi / info["n_phi"]
    nr, nc = info["n_theta_fine"] // 2, info["n_phi"]
    cells = rng.permutation(nr * nc)
    count = np.resize(COUNTS, len(cells))
    cell = np.repeat(cells, count)
    assert len(cell) >= n
    cell = cell[:n]
    p = np.stack([(cell // nc + rng.uniform(0.01, 0.99, n)) * hth, (cell % nc + rng.uniform(0.01, 0.99, n)) * hph,
                  rng.uniform(0, 2 * np.pi, n)], 1)
    p[0], p[-1] = [0.0, 1.0, 0.3], [np.pi, 2.0, 0.4]
    return np.ascontiguousarray(p[rng.permutation(n)])


def _gradients(plan, a, b, p, y):
    plan.enable_timing(True)
    g = plan.adjoint(b, p, y), plan.adjoint_beam(a, p, y)
    binned = plan.stage_times()["binning"][1]
    plan.enable_timing(False)
    return [v.cpu().numpy() for v in g], binned


@pytest.mark.parametrize("width,kmax,n", [
    (14, 0, 3001), (14, 7, 4096), (14, 15, 4096), (16, 1, 4095), (12, 8, 4000), (10, 16, 4096), (8, 15, 4096),
    (6, 23, 4096), (14, 23, 4096), (16, 39, 2000),
    (4, 0, 100_000), (4, 15, 30_000), (6, 1, 50_000), (8, 7, 20_000), (10, 3, 20_000), (12, 6, 6000), (14, 0, 9000),
    (14, 0, 2000), (14, 1, 30_001), (14, 7, 8191), (14, 15, 4097), (14, 16, 5000), (16, 15, 4500), (16, 23, 4097)])
def test_binned_scatter_matches_the_per_sample_path(monkeypatch, width, kmax, n):
    L = 48
    a = torch.from_numpy(W.sky_alm(L, 41)).cuda()
    b = torch.from_numpy(W.beam_alm(L, kmax, 42, kind="flat")).cuda()
    plan = api.Plan(L, kmax, "fp64", kernel_width=width)
    monkeypatch.setenv("SC_GATHER_PATH", "direct")
    direct = api.Plan(L, kmax, "fp64", kernel_width=width)
    monkeypatch.delenv("SC_GATHER_PATH")
    p = torch.from_numpy(_pointings(plan.info(), n, 43 + n)).cuda()
    y = torch.from_numpy(np.random.default_rng(44).standard_normal(n)).cuda()
    got, binned = _gradients(plan, a, b, p, y)
    ref, none = _gradients(direct, a, b, p, y)
    assert binned == 2 and none == 0
    for g, r in zip(got, ref):
        assert np.max(np.abs(g - r)) <= 1e-12 * np.max(np.abs(r))


@pytest.mark.parametrize("width,kmax,n", [(14, 0, 1500), (14, 0, 4097), (14, 1, 5000), (4, 0, 20_000), (8, 3, 4096)])
def test_small_passes_are_not_binned(width, kmax, n):
    L = 48
    a = torch.from_numpy(W.sky_alm(L, 41)).cuda()
    b = torch.from_numpy(W.beam_alm(L, kmax, 42, kind="flat")).cuda()
    plan = api.Plan(L, kmax, "fp64", kernel_width=width)
    p = torch.from_numpy(_pointings(plan.info(), n, 45)).cuda()
    y = torch.from_numpy(np.random.default_rng(44).standard_normal(n)).cuda()
    assert _gradients(plan, a, b, p, y)[1] == 0
