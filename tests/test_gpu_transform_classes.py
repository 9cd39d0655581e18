"""The runtime-planned transforms at the edges of their thread-count classes (576 and 1152
points), forward against the oracle and adjoint by the dot product.

Tolerances as for the other transform lengths: the FP64 form (W = 14) reaches the
convolution to about 1e-13, so 1e-11; the adjoint is the exact transpose up to rounding.
"""
import numpy as np
import pytest
import torch

import oracle
import workloads as W
from parity import assert_parity
from paper_2201_03478_amd import api

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [134, 138, 142, 145, 150, 270, 278, 286, 290, 300])
def test_transform_class_edges(L):
    K, n = 3, 300
    a, b = W.sky_alm(L, 81), W.beam_alm(L, K, 82)
    p = W.uniform_pointings(n, 83)
    ta, tb, tp = (torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (a, b, p))
    plan = api.Plan(L, K, "fp64")
    tod = plan.convolve(ta, tb, tp)
    inf = plan.info()
    assert_parity(tod.cpu().numpy(), oracle.convolve(a, b, L, K, p), 1e-11,
                  "L=%d lengths %d/%d/%d" % (L, inf["n_fft_theta"], inf["n_theta_fine"], inf["n_phi"]))
    y = torch.from_numpy(np.random.default_rng(84).standard_normal(n)).cuda()
    g = plan.adjoint(tb, tp, y)
    lhs, rhs = float((y * tod).sum()), float((g.real * ta.real + g.imag * ta.imag).sum())
    assert abs(lhs - rhs) <= 1e-11 * float(y.norm() * tod.norm())
