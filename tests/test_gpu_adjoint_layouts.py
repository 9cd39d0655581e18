"""The adjoints at every ring layout and at the transform lengths with kernels of their own.

Entries of the gradients one by one: with e the unit sky (or beam) of one coefficient, Re or
Im, <y, A e> from the forward path is that part of the gradient's entry.  Both sides are sums
of the same FP64 terms in other orders; the forward path reaches 1e-12 of the largest datum, so
1e-11 of sum |y| max |A e| bounds the difference with room for the adjoint's own rounding.
"""
import numpy as np
import pytest
import torch

import workloads as W
from paper_2201_03478_amd import api

pytestmark = pytest.mark.gpu


def _index(lmax, l, m):
    return m * (2 * lmax + 1 - m) // 2 + l


def _check(L, K, n, seed, prec="fp64", bar=1e-11):
    a, b = (torch.from_numpy(v).cuda() for v in (W.sky_alm(L, seed), W.beam_alm(L, K, seed + 1, kind="flat")))
    p_np = W.uniform_pointings(n, seed + 2)
    p_np[0, 0], p_np[1, 0], p_np[2, 1], p_np[3, 1] = 0.0, np.pi, 0.0, 6.283185307179586
    p = torch.from_numpy(p_np).cuda()
    plan = api.Plan(L, K, prec)
    y = torch.from_numpy(np.random.default_rng(seed + 3).standard_normal(n)).cuda().to(plan.tod_dtype)
    g, h = plan.adjoint(b, p, y), plan.adjoint_beam(a, p, y)
    sky = [(0, 0), (L, 0), (L, L), (L, 1), (L - 1, L // 2), (L // 2, L // 3), (K, K), (K + 1, K)]
    beam = [(0, 0), (L, 0), (L, K), (K, K), (L // 2, K // 2), (L - 1, max(K - 1, 0))]
    for grad, pairs, size in ((g, sky, a.numel()), (h, beam, b.numel())):
        for l, m in pairs:
            i = _index(L, l, m)
            for part in (1.0, 1j) if m > 0 else (1.0,):
                e = torch.zeros(size, dtype=torch.complex128, device="cuda")
                e[i] = part
                d = plan.convolve(e, b, p) if grad is g else plan.convolve(a, e, p)
                d, yy = d.double(), y.double()
                want = float((d * yy).sum())
                got = float(grad[i].real if part == 1.0 else grad[i].imag)
                scale = float(d.abs().max() * yy.abs().sum())
                assert abs(got - want) <= bar * scale, (l, m, part, got, want, scale)


# northern rings 16, 32, 54, ... : 1 to 9 rings per lane of one wave, then two and four waves
@pytest.mark.parametrize("L", [30, 63, 107, 150, 200, 255, 290, 330, 383, 410, 480, 530, 640, 720, 1150])
def test_every_ring_layout(L):
    _check(L, 2, 200, 11)


# phi lengths 1080, 2160 and 4320 (two k at a time: even and odd counts), theta 540/1080 to 2160/4320
@pytest.mark.parametrize("kmax", [0, 1, 2, 3])
@pytest.mark.parametrize("L", [256, 269, 512, 539, 1024, 1079])
def test_lengths_with_their_own_kernels(L, kmax):
    info = api.Plan(L, kmax, "fp64").info()
    assert info["n_phi"] in (1080, 2160, 4320) and info["n_theta_fine"] == info["n_phi"]
    _check(L, kmax, 200, 21)


@pytest.mark.parametrize("prec", ["f64maps_f32gather", "mixed"])
@pytest.mark.parametrize("L,kmax", [(256, 2), (256, 3), (512, 2), (512, 3), (1024, 1), (1024, 2)])
def test_lengths_with_their_own_kernels_fp32(prec, L, kmax):
    """FP32 maps and scatter: 2^-24 in the maps, products and sums, a few hundred terms."""
    _check(L, kmax, 200, 31, prec, 1e-5)
