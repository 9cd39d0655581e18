"""Rounding of the runtime-planned transforms' twiddles, emulated in float64.

A pass of radix R multiplies by w^r, r < R.  The kernels load w, w^2, w^4 and w^8 and form
w^r = w^{r mod 4} w^{4 (r / 4)} with w^3 = w w^2 and w^12 = w^4 w^8: at most three rounded
products, each of relative error below 2 x 2^-53 against a transform's 8 x 2^-53 or more, so
the transform's error may grow by a tenth at most over loading every w^r.  (Powers of w alone
carry w's own rounding r times: up to twice the error.)
"""
import numpy as np
import pytest

LD, CL = np.longdouble, np.clongdouble
TWO_PI = LD("6.28318530717958647692528676655900576839")


def _cis(x, ct):
    return (np.cos(TWO_PI * x) + 1j * np.sin(TWO_PI * x)).astype(ct)


def _twiddles(frac, radix, how, ct):
    if how == "loaded":
        return [_cis(-frac * r, ct) for r in range(radix)]
    if how == "powers":
        w = [np.ones_like(frac, ct), _cis(-frac, ct)]
        for r in range(2, radix):
            w.append(w[r - 2] * (w[1] * w[1]) if r > 2 else w[1] * w[1])
        return w
    w1, w2, w4, w8 = (_cis(-frac * b, ct) for b in (1, 2, 4, 8))
    lo, hi = [None, w1, w2, w1 * w2], [None, w4, w8, w4 * w8]
    return [np.ones_like(w1)] + [lo[r % 4] if r < 4 else hi[r // 4] if r % 4 == 0 else hi[r // 4] * lo[r % 4]
                                 for r in range(1, radix)]


def _transform(x, radices, how, ct):
    n, ns, buf = len(x), 1, x.astype(ct)
    for radix in radices:
        nb = n // radix
        j = np.arange(nb)
        k, g = j % ns, j // ns
        v = np.stack([buf[j + r * nb] for r in range(radix)])
        if ns > 1:
            v = v * np.stack(_twiddles(k.astype(LD) / LD(ns * radix), radix, how, ct))
        i = np.arange(radix)
        y = _cis(-LD(1) * (np.outer(i, i) % radix) / LD(radix), ct) @ v
        buf = np.empty(n, ct)
        for r in range(radix):
            buf[g * ns * radix + k + r * ns] = y[r]
        ns *= radix
    return buf


@pytest.mark.parametrize("radices", [(16, 9, 4), (16, 5, 5, 3), (16, 16, 5, 4), (16, 16, 16, 2), (9, 5, 5, 5, 8),
                                     (10, 12, 15), (16, 16, 5, 8)])
def test_products_of_four_loads_keep_the_error(radices):
    n = int(np.prod(radices))
    rng = np.random.default_rng(n)
    x = rng.standard_normal(n) + 1j * rng.standard_normal(n)
    ref = _transform(x, radices, "loaded", CL)
    assert np.abs(ref - np.fft.fft(x)).max() <= 1e-12 * np.abs(ref).max()
    err = {h: float(np.sqrt(np.mean(np.abs(_transform(x, radices, h, np.complex128) - ref) ** 2)))
           for h in ("loaded", "products", "powers")}
    assert err["products"] <= 1.1 * err["loaded"]
    assert err["powers"] > err["products"]
