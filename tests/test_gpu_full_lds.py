"""Transforms of 9217 to 10240 points (lmax 2304 to 2559), one workgroup's whole LDS.

At lmax 2559 all three lengths sit at the limit (5120, 10240, 10240), at 2560 the split
stages take over.  Against the oracle's direct sum, with the bars of the band limits around
them: 1e-11 for the FP64 form, 1e-6 for the FP32-map form; and the adjoints' dot products to
1e-11 in FP64.
"""
import numpy as np
import pytest
import torch

import workloads as W
from paper_2201_03478_amd import api
from parity import assert_parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,bar", [("fp64", 1e-11), ("f64maps_f32gather", 1e-6)])
@pytest.mark.parametrize("L", [2304, 2500, 2559, 2560])
def test_full_lds_transforms(oracle_lib, L, prec, bar):
    K = 1
    a_np, b_np = W.sky_alm(L, 71), W.beam_alm(L, K, 72, kind="flat")
    b_np[:L + 1] = b_np[:L + 1].real
    p_np = W.uniform_pointings(12, 73)
    p_np[0], p_np[1] = [0.0, 0.4, 1.3], [np.pi, 2.2, 0.1]
    a, b, p = (torch.from_numpy(v).cuda() for v in (a_np, b_np, p_np))
    plan = api.Plan(L, K, prec)
    assert (plan.info()["n_theta_fine"] <= 10240) == (L < 2560)
    tod = plan.convolve(a, b, p)
    assert_parity(tod.double().cpu().numpy(), oracle_lib.convolve(a_np, b_np, L, K, p_np), bar, "lmax %d %s" % (L, prec))
    if prec == "fp64":
        y = torch.from_numpy(np.random.default_rng(74).standard_normal(12)).cuda()
        lhs = float(torch.dot(tod, y))
        for g, x in ((plan.adjoint(b, p, y), a), (plan.adjoint_beam(a, p, y), b)):
            assert abs(lhs - float((g.conj() * x).real.sum())) <= 1e-11 * abs(lhs)
