"""The recursion without its coefficient table (which plans above 8 GiB of it do not have).

The kernels then form the coefficients of each chunk of 64 steps as the table's kernel does, up
to the compiler's choice of fused operations (a relative 2^-53 per coefficient, over at most
384 steps), and the gradients' scatter adds with atomics in any order (at most a few hundred
additions of the same error): 1e-12 of the largest value bounds both.  Columns of one step, of
a step more or less than a group (4 and 16 steps) and a chunk (64), and ones of several chunks.
"""
import pytest
import torch

import workloads as W
from paper_2201_03478_amd import api

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,K", [(0, 0), (1, 1), (3, 2), (4, 1), (15, 3), (16, 15), (63, 5), (64, 64), (65, 2),
                                 (127, 4), (130, 12), (260, 3), (384, 12)])
def test_without_table(monkeypatch, L, K):
    a, b = (torch.from_numpy(v).cuda() for v in (W.sky_alm(L, 1), W.beam_alm(L, K, 2, kind="flat")))
    p_np = W.uniform_pointings(200, 3)
    p_np[0, 0], p_np[1, 0] = 0.0, 3.141592653589793
    p = torch.from_numpy(p_np).cuda()
    y = torch.randn(200, dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(4))
    table = api.Plan(L, K, "fp64")
    monkeypatch.setenv("SC_REC_TABLE", "0")
    none = api.Plan(L, K, "fp64")
    monkeypatch.delenv("SC_REC_TABLE")
    assert none.info()["workspace_bytes"] < table.info()["workspace_bytes"]
    for g, h in ((none.convolve(a, b, p), table.convolve(a, b, p)), (none.adjoint(b, p, y), table.adjoint(b, p, y)),
                 (none.adjoint_beam(a, p, y), table.adjoint_beam(a, p, y))):
        assert float((g - h).abs().max()) <= 1e-12 * float(h.abs().max())
