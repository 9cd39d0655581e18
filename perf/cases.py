"""Workloads whose time is followed, each through the package's public entry points.

A case is a dict of plain values.  "kind" names the call:
  convolve     Plan.convolve: new sky and beam, map synthesis, then the TOD
  interpolate  Plan.interpolate: the TOD of new pointings from resident maps
  gradient     sidelobe_convolve and its backward pass (TOD and sky gradient)
  beam         Plan.adjoint_beam: the beam gradient of a residual
  psi          Plan.build_psi_cube and Plan.interpolate_psi from resident maps
  batch        Batch.run: detectors of different sizes sharing one sky
  dipole       dipole_response: orbital dipole and quadrupole through the beam
Skies are Gaussian with C_l = 1/(l(l+1)), beams sidelobe-like ((1+k)^-1.5 exp(-l/200)),
pointings a 1 rpm circular scan sampled at 32.5 Hz ("scan") or uniform ("uniform").

exact() evaluates the same quantities in 64 bits without the package: the three-dimensional
Fourier coefficients of the convolution from Wigner's d at pi/2, then non-uniform Fourier
evaluation at the pointings.
"""
import math

import numpy as np
import torch

from paper_2201_03478_amd import api

DEV = "cuda" if torch.cuda.is_available() else "cpu"

# One detector of a batch: (lmax, kmax, share of the batch's samples).
BATCH_DETECTORS = [(1024, 32, 0.34), (512, 100, 0.25), (256, 100, 0.2), (512, 32, 0.15), (256, 8, 0.05),
                   (1024, 8, 0.01)]


def listed():
    f32, f64 = "f64maps_f32gather", "fp64"
    return [
        # The smallest whole call: a low-resolution FP64 check of a beam model.
        dict(name="tiny-fp64", kind="convolve", precision=f64, lmax=64, kmax=4, n=100_000, pointing="uniform"),
        # Serving: one minute of scan (1 rpm at 32.5 Hz) from resident maps; latency and launches count.
        dict(name="minute", kind="interpolate", precision=f32, lmax=256, kmax=8, n=1950, pointing="scan"),
        # The headline: sidelobe beam at lmax 512, mmax 100, 1e7 scan samples, new sky and beam.
        dict(name="sidelobe", kind="convolve", precision=f32, lmax=512, kmax=100, n=10_000_000, pointing="scan"),
        # More pointing from the same maps (a ragged stretch of scan).
        dict(name="sidelobe-tod", kind="interpolate", precision=f32, lmax=512, kmax=100, n=3_333_337,
             pointing="scan"),
        # Accuracy runs: FP64 maps and interpolation at the default width (1e-12).
        dict(name="fp64", kind="convolve", precision=f64, lmax=384, kmax=45, n=1_000_003, pointing="scan"),
        # Many samples of a narrow beam at high resolution, mixed-precision synthesis.
        dict(name="precision", kind="convolve", precision="mixed", lmax=1024, kmax=16, n=100_000_000,
             pointing="scan"),
        # One optimisation step of the sky: forward and backward through autograd.
        dict(name="gradient", kind="gradient", precision=f32, lmax=512, kmax=32, n=10_000_000, pointing="scan"),
        # Beam fit in FP64 on a small problem.
        dict(name="beam-fp64", kind="beam", precision=f64, lmax=128, kmax=8, n=200_000, pointing="scan"),
        # Second step on a psi grid: cube from resident maps, then three-dimensional interpolation.
        dict(name="psi-cube", kind="psi", precision=f32, lmax=512, kmax=100, n=2_000_003, pointing="scan"),
        # Six detectors of one sky in one replayed graph.
        dict(name="batch", kind="batch", precision=f32, lmax=1024, kmax=100, n=6_000_000, pointing="scan"),
        # The top of the band-limit range: transforms longer than one workgroup holds.
        dict(name="high-lmax", kind="convolve", precision=f32, lmax=2500, kmax=4, n=1_000_000, pointing="scan"),
        # Orbital dipole of a day's samples.
        dict(name="dipole", kind="dipole", precision=f64, lmax=512, kmax=100, n=10_000_000, pointing="scan"),
    ]


def draw(rng):
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    top = [work(c) for c in listed()]
    most = {k: max(w[k] for w in top) for k in ("bytes", "flops")}
    while True:
        kind = rng.choice(["convolve", "convolve", "convolve", "interpolate", "interpolate", "gradient", "beam", "psi",
                           "batch", "dipole"])
        precision = {"psi": "f64maps_f32gather", "batch": "f64maps_f32gather", "dipole": "fp64"}.get(
            kind, rng.choice(["f64maps_f32gather", "f64maps_f32gather", "mixed", "fp64"]))
        f64 = precision == "fp64" and kind != "dipole"
        lmax = size(32, 512 if f64 or kind == "psi" else 1024)
        kmax = min(lmax, size(1, 45 if f64 else 100))
        if kind == "convolve" and not f64 and rng.random() < 0.2:
            lmax, kmax = size(1024, 2500), rng.randint(0, 4)
        hi = {"gradient": 10_000_000, "beam": 10_000_000, "psi": 10_000_000, "batch": 6_000_000}.get(kind, 30_000_000)
        n = size(1000, 1_000_000 if f64 else hi)
        case = dict(kind=kind, precision=precision, lmax=lmax, kmax=kmax, n=n,
                    pointing=rng.choice(["scan", "scan", "uniform"]) if n <= 1_000_000 else "scan")
        w = work(case)
        if w["bytes"] <= most["bytes"] and w["flops"] <= most["flops"]:
            return case


# ---------------------------------------------------------------- inputs

def _n_alm(lmax, mmax):
    return (mmax + 1) * (lmax + 1) - mmax * (mmax + 1) // 2


def _lm(lmax, mmax):
    """(l, m) of each entry of a triangular m-major array."""
    m = torch.cat([torch.full((lmax + 1 - i,), i, device=DEV) for i in range(mmax + 1)])
    start = torch.tensor([_n_alm(lmax, i - 1) - i if i else 0 for i in range(mmax + 1)], device=DEV)
    return torch.arange(m.numel(), device=DEV) - start[m], m


def _gauss(n, g):
    return torch.randn(n, 2, dtype=torch.float64, device=DEV, generator=g)


def _sky(lmax, g):
    l, m = _lm(lmax, lmax)
    cl = torch.where(l > 0, 1.0 / (l * (l + 1.0)).clamp(min=1.0), 0.0)
    x = _gauss(l.numel(), g) * (cl * torch.where(m > 0, 0.5, 1.0)).sqrt()[:, None]
    x[:, 1] *= m > 0
    return torch.view_as_complex(x)


def _beam(lmax, kmax, g):
    l, k = _lm(lmax, kmax)
    x = _gauss(l.numel(), g) * ((1.0 + k) ** -1.5 * torch.exp(-l / 200.0) / torch.where(k > 0, 2.0, 1.0).sqrt())[:, None]
    x[:, 1] *= k > 0
    return torch.view_as_complex(x)


def _scan(n, t0, psi0):
    """1 rpm circles of 85 deg opening about an ecliptic spin axis moving 1 deg/day, 32.5 Hz."""
    out = torch.empty(n, 3, dtype=torch.float64, device=DEV)
    alpha, rate, spin = math.radians(85.0), math.radians(1.0) / 86400.0, 2.0 * math.pi / 60.0
    for s in range(0, n, 1 << 23):
        t = t0 + torch.arange(s, min(n, s + (1 << 23)), dtype=torch.float64, device=DEV) / 32.5
        lam, w = rate * t, spin * t
        cl, sl, cw, sw = lam.cos(), lam.sin(), w.cos(), w.sin()
        ca, sa = math.cos(alpha), math.sin(alpha)
        x, y, z = ca * cl - sa * sw * sl, ca * sl + sa * sw * cl, sa * cw
        vx = -ca * rate * sl - sa * (spin * cw * sl + sw * rate * cl)
        vy = ca * rate * cl + sa * (spin * cw * cl - sw * rate * sl)
        vz = -sa * spin * sw
        theta, phi = torch.arccos(z.clamp(-1, 1)), torch.remainder(torch.arctan2(y, x), 2 * math.pi)
        ct, st, cp, sp = theta.cos(), theta.sin(), phi.cos(), phi.sin()
        psi = torch.arctan2(vy * cp - vx * sp, vx * ct * cp + vy * ct * sp - vz * st)
        out[s:s + t.numel()] = torch.stack([theta, phi, torch.remainder(psi + psi0, 2 * math.pi)], 1)
    return out


def _pointings(case, n, g, t0, psi0):
    if case["pointing"] == "scan":
        return _scan(n, t0, psi0)
    u = torch.rand(n, 3, dtype=torch.float64, device=DEV, generator=g)
    return torch.stack([torch.arccos(2 * u[:, 0] - 1), 2 * math.pi * u[:, 1], 2 * math.pi * u[:, 2]], 1)


def _detectors(case):
    """(lmax, kmax, n) of a batch's detectors, scaled to the case's largest lmax and kmax."""
    out = []
    for l, k, share in BATCH_DETECTORS:
        lmax = max(1, l * case["lmax"] // 1024)
        out.append((lmax, min(lmax, max(1, k * case["kmax"] // 100)), max(1, int(share * case["n"]))))
    return out


def _inputs(case, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    L, K, n = case["lmax"], case["kmax"], case["n"]
    u = torch.rand(2, dtype=torch.float64, device=DEV, generator=g).tolist()
    t0, psi0 = 86400.0 * 365 * u[0], 2 * math.pi * u[1]
    x = dict(alm=_sky(L, g))
    if case["kind"] == "batch":
        x["dets"] = [dict(lmax=l, kmax=k, blm=_beam(l, k, g), ptg=_pointings(case, m, g, t0 + 1000.0 * i, psi0 + i))
                     for i, (l, k, m) in enumerate(_detectors(case))]
        return x
    x["blm"] = _beam(L, K, g)
    x["ptg"] = _pointings(case, n, g, t0, psi0)
    if case["kind"] in ("gradient", "beam"):
        x["y"] = torch.randn(n, dtype=torch.float64 if case["precision"] == "fp64" else torch.float32, device=DEV,
                             generator=g)
    if case["kind"] == "dipole":
        x["period"] = 1950 * 45  # samples per pointing period: 45 minutes
        x["beta"] = 1e-4 * torch.randn(-(-n // x["period"]), 3, dtype=torch.float64, device=DEV, generator=g)
        x["T0"], x["q"] = 2.7255, 1.3
    return x


# ---------------------------------------------------------------- the calls

def prepare(case, seed):
    s = _inputs(case, seed)
    s["kind"] = case["kind"]
    if case["kind"] == "batch":
        s["batch"] = api.Batch(s["dets"], case["lmax"], case["precision"])
    elif case["kind"] == "dipole":
        s["lmax"], s["kmax"] = case["lmax"], case["kmax"]
    else:
        s["plan"] = api.Plan(case["lmax"], case["kmax"], case["precision"])
        if case["kind"] in ("interpolate", "psi"):
            s["plan"].set_sky_beam(s["alm"], s["blm"])
    return s


def run(s):
    kind = s["kind"]
    if kind == "convolve":
        return s["plan"].convolve(s["alm"], s["blm"], s["ptg"])
    if kind == "interpolate":
        return s["plan"].interpolate(s["ptg"])
    if kind == "gradient":
        alm = s["alm"].detach().requires_grad_()
        tod = api.sidelobe_convolve(alm, s["blm"], s["ptg"], s["plan"])
        tod.backward(s["y"])
        return [tod.detach(), alm.grad]
    if kind == "beam":
        return s["plan"].adjoint_beam(s["alm"], s["ptg"], s["y"])
    if kind == "psi":
        s["plan"].build_psi_cube()
        return s["plan"].interpolate_psi(s["ptg"])
    if kind == "batch":
        return s["batch"].run(s["alm"], use_graph=True)
    return api.dipole_response(s["blm"], s["lmax"], s["kmax"], s["ptg"], s["beta"], s["period"], s["T0"], s["q"])


def _synthesis(L, K):
    """Operations of the maps of every k <= K: 12 per d value on northern rings, then the transforms."""
    d = sum(L + 1 - max(m, k) for k in range(K + 1) for m in (range(0, L + 1) if L < 200 else range(0, L + 1, 8)))
    d *= (1 if L < 200 else 8) * (L + 1)
    fft = (K + 1) * 5.0 * (2 * L * 4 * L * math.log2(4 * L + 2) + 2 * L * 4 * L * math.log2(4 * L + 2))
    return 12.0 * d + fft


def work(case):
    L, K, n, kind = case["lmax"], case["kmax"], case["n"], case["kind"]
    W, out = (14, 8) if case["precision"] == "fp64" else (8, 4)
    ab = 16.0 * (_n_alm(L, L) + _n_alm(L, K))
    if kind == "batch":
        dets = _detectors(case)
        return {"bytes": ab + sum(16.0 * _n_alm(l, k) + 28.0 * m for l, k, m in dets),
                "flops": sum(_synthesis(l, k) + 2.0 * (2 * k + 1) * W * W * m for l, k, m in dets)}
    taps = 2.0 * (2 * K + 1) * W * W * n
    maps = 2.0 * out * (2 * K + 1) * 4 * L * L
    if kind == "convolve":
        return {"bytes": ab + (24.0 + out) * n, "flops": _synthesis(L, K) + taps}
    if kind == "interpolate":  # the maps, or as much of them as the samples' stencils cover
        return {"bytes": (24.0 + out) * n + min(maps, out * (2 * K + 1) * W * W * float(n)), "flops": taps}
    if kind == "gradient":
        return {"bytes": ab + 16.0 * _n_alm(L, L) + (24.0 + 2 * out) * n, "flops": 2 * (_synthesis(L, K) + taps)}
    if kind == "beam":
        return {"bytes": ab + 16.0 * _n_alm(L, K) + (24.0 + out) * n, "flops": _synthesis(L, K) + taps}
    if kind == "psi":
        return {"bytes": maps + (24.0 + out) * n, "flops": 20.0 * L * L * (2 * K + 1) * math.log2(2 * K + 4)
                + 2.0 * W ** 3 * n}
    return {"bytes": 32.0 * n, "flops": 60.0 * n}


# ---------------------------------------------------------------- the same in 64 bits

def _dense(x, L, M):
    """[l, m] matrix of a triangular array (zero where l < m)."""
    l, m = _lm(L, M)
    full = torch.zeros(L + 1, M + 1, dtype=torch.complex128, device=DEV)
    full = full.index_put((l, m), x)
    return torch.cat([torch.complex(full[:, :1].real, torch.zeros_like(full[:, :1].real)), full[:, 1:]], 1)


def _deltas(L, n, m):
    """d^l_{nm}(pi/2) for l = 0 .. L, [l, n, m]; values carried as mantissa and binary exponent."""
    n, m = n[:, None].double(), m[None, :].double()
    l0, lo = torch.maximum(n, m), torch.minimum(n, m)
    lg = torch.tensor(np.concatenate([[0.0], np.cumsum(np.log2(np.arange(1, 2 * L + 2).astype(np.longdouble)))])
                      .astype(np.float64), device=DEV)  # log2 of factorials, summed in extended precision
    e = 0.5 * (lg[(2 * l0).long()] - lg[(l0 + lo).long()] - lg[(l0 - lo).long()]) - l0
    E = e.floor()
    first = torch.exp2(e - E) * torch.where((n > m) & ((n - m) % 2 == 1), -1.0, 1.0)
    out = torch.zeros(L + 1, l0.shape[0], l0.shape[1], dtype=torch.float64, device=DEV)
    u, v = torch.zeros_like(e), torch.zeros_like(e)  # values at l and l - 1
    for l in range(L + 1):
        if l:
            j = l - 1.0
            nm = (l * l - n * n).clamp(min=0.0).sqrt() * (l * l - m * m).clamp(min=0.0).sqrt()
            below = ((j * j - n * n).clamp(min=0.0) * (j * j - m * m).clamp(min=0.0)).sqrt()
            step = -(2 * j + 1) * (n * m / j if j else 0.0) * u - l * below / max(j, 1.0) * v
            new = torch.where(l > l0, step / nm.clamp(min=1e-300), 0.0)
            u, v = new, u
        u = torch.where(l0 == l, first, u)
        big = u.abs() > 2.0 ** 300
        u, v, E = torch.where(big, u * 2.0 ** -300, u), torch.where(big, v * 2.0 ** -300, v), E + 300.0 * big
        out[l] = u * torch.exp2(E)
    return out


def _coefficients(a, b, L, K):
    """C[n, m, k], |n|, |m| <= L (both wrapped): c = sum_k f_k Re e^{ik psi} sum C e^{i(n theta + m phi)}."""
    m, k, l = torch.arange(L + 1, device=DEV), torch.arange(K + 1, device=DEV), torch.arange(L + 1, device=DEV)
    am = a * torch.where(m % 2 == 0, 1.0, -1.0)
    alt = torch.where(l % 2 == 0, 1.0, -1.0)[:, None]
    pos, neg = [], []
    block = max(1, min(L + 1, int(2e9 / (8.0 * (L + 1) ** 2))))
    for n0 in range(0, L + 1, block):
        ns = torch.arange(n0, min(L + 1, n0 + block), device=DEV)
        d = _deltas(L, ns, m)
        for i in range(ns.numel()):
            s = 1.0 if (n0 + i) % 2 == 0 else -1.0
            right = b.conj() * d[:, i, :K + 1]
            pos.append((a * d[:, i]).transpose(0, 1).contiguous() @ right)
            neg.append((am.conj() * d[:, i] * (alt * s)).transpose(0, 1).contiguous() @ right)
    c = torch.cat([torch.stack(pos), torch.stack(neg)[:, 1:].flip(1)], 1)  # n >= 0; m = 0 .. L, -L .. -1
    mm = torch.cat([m, m[1:].flip(0).neg()])
    odd = torch.where((mm[:, None] + k[None, :]) % 2 == 0, 1.0, -1.0)
    quarter = torch.tensor([1, 1j, -1, -1j], dtype=torch.complex128, device=DEV)
    phase = quarter[(k[None, :] - mm[:, None]) % 4]
    return torch.cat([c, c[1:].flip(0) * odd], 0) * phase


def _smooth(n):
    while True:
        r = n
        for p in (2, 3, 5):
            while r % p == 0:
                r //= p
        if r == 1 and n % 2 == 0:
            return n
        n += 1


def _kernel(x, W):
    z = (x * (2.0 / W)) ** 2
    return torch.where(z < 1, torch.exp(2.3 * W * ((1 - z).clamp(min=0.0).sqrt() - 1)), 0.0)


def _grid(C, L, W):
    """The oversampled grid [theta, phi, k] whose kernel interpolation gives the Fourier series."""
    N = _smooth(max(4 * L + 4, 4 * W))
    x, w = np.polynomial.legendre.leggauss(400)
    t = np.pi / 2 * x  # z = sin t removes the square root's end points
    wave = torch.cat([torch.arange(L + 1, device=DEV), torch.arange(-L, 0, device=DEV)])
    z = torch.tensor(np.sin(t), device=DEV)
    wt = torch.tensor(w * np.pi / 2 * np.cos(t) * np.exp(2.3 * W * (np.cos(t) - 1)) * W / 2, device=DEV)
    hat = (torch.cos(2 * math.pi / N * wave.double()[:, None] * (W / 2) * z[None, :]) * wt).sum(1)
    at = wave % N
    out = []
    for k in range(C.shape[2]):
        f = torch.zeros(N, N, dtype=torch.complex128, device=DEV)
        f = f.index_put((at[:, None], at[None, :]), C[:, :, k] / (hat[:, None] * hat[None, :]))
        out.append(torch.fft.ifft2(f) * (N * N))
    return out, N


def _taps(ptg, N, W):
    """Cell index and weight of each of the W x W taps of each pointing."""
    step = 2 * math.pi / N
    at, wt = [], []
    for x in (ptg[:, 0] / step, ptg[:, 1] / step):
        i = torch.floor(x).long() - W // 2 + 1
        i = i[None, :] + torch.arange(W, device=DEV)[:, None]
        at.append(i % N)
        wt.append(_kernel(x[None, :] - i, W))
    for p in range(W):
        for q in range(W):
            yield at[0][p] * N + at[1][q], wt[0][p] * wt[1][q]


def _fold(psi, K):
    k = torch.arange(K + 1, dtype=torch.float64, device=DEV)
    e = torch.polar((k > 0).double() + 1, torch.zeros_like(k))
    return e * torch.polar(torch.ones(1, dtype=torch.float64, device=DEV), psi[:, None] * k)


def _evaluate(maps, N, K, ptg, W):
    flat = torch.view_as_real(torch.stack(maps, 2).reshape(N * N, K + 1)).reshape(N * N, 2 * K + 2)
    out = torch.empty(ptg.shape[0], dtype=torch.float64, device=DEV)
    chunk = max(1024, int(1e9 / (16 * (K + 1))))
    for s in range(0, ptg.shape[0], chunk):
        p = ptg[s:s + chunk]
        acc = torch.zeros(p.shape[0], 2 * K + 2, dtype=torch.float64, device=DEV)
        for at, wt in _taps(p, N, W):
            acc.addcmul_(flat.index_select(0, at), wt[:, None])
        t = torch.view_as_complex(acc.view(-1, K + 1, 2))
        out[s:s + chunk] = (t * _fold(p[:, 2], K)).real.sum(1)
    return out


def _spread(N, K, ptg, y, W):
    flat = torch.zeros(N * N, 2 * K + 2, dtype=torch.float64, device=DEV)
    chunk = max(1024, int(1e9 / (16 * (K + 1))))
    for s in range(0, ptg.shape[0], chunk):
        p = ptg[s:s + chunk]
        v = torch.view_as_real(_fold(p[:, 2], K).conj().resolve_conj() * y[s:s + chunk, None]).reshape(-1, 2 * K + 2)
        for at, wt in _taps(p, N, W):
            flat.index_add_(0, at, v * wt[:, None])
    return torch.view_as_complex(flat.view(N, N, K + 1, 2))


def exact(case, seed):
    x = _inputs(case, seed)
    L, K, kind = case["lmax"], case["kmax"], case["kind"]
    W = 14 if case["precision"] == "fp64" else 10
    if kind == "dipole":
        return _dipole(case, x)
    if kind == "batch":
        sky, out = _dense(x["alm"], L, L), []
        for d in x["dets"]:
            l, k = d["lmax"], d["kmax"]
            maps, N = _grid(_coefficients(sky[:l + 1, :l + 1], _dense(d["blm"], l, k), l, k), l, W)
            out.append(_evaluate(maps, N, k, d["ptg"], W))
        return out
    back = kind in ("gradient", "beam")
    a, b = x["alm"].clone().requires_grad_(kind == "gradient"), x["blm"].clone().requires_grad_(kind == "beam")
    if back and (L > 600 or (2 * L + 2.0) ** 2 * 4 * (K + 1) * 16 > 1e10):
        return None  # too large to hold every factor of the coefficients
    if 1e-9 * (case["n"] * 1.0) * W * W * (K + 1) > 300:
        return None  # too long
    with torch.set_grad_enabled(back):
        maps, N = _grid(_coefficients(_dense(a, L, L), _dense(b, L, K), L, K), L, W)
    if not back:
        return _evaluate(maps, N, K, x["ptg"], W)
    g = _spread(N, K, x["ptg"], x["y"].double(), W)
    grad, = torch.autograd.grad(maps, [a if kind == "gradient" else b], [g[:, :, k].contiguous() for k in range(K + 1)])
    if kind == "beam":
        return grad
    return [_evaluate([m.detach() for m in maps], N, K, x["ptg"], W), grad]


def _dipole(case, x):
    b = _dense(x["blm"][:], case["lmax"], case["kmax"])
    q = lambda l, k: b[l, k] if l <= case["lmax"] and k <= min(l, case["kmax"]) else torch.zeros_like(b[0, 0])
    pi = math.pi
    S = torch.stack([-math.sqrt(8 * pi / 3) * q(1, 1).real, math.sqrt(8 * pi / 3) * q(1, 1).imag,
                     math.sqrt(4 * pi / 3) * q(1, 0).real])
    tr, zz = math.sqrt(4 * pi) * q(0, 0).real / 3, math.sqrt(16 * pi / 5) * q(2, 0).real / 3
    c = math.sqrt(8 * pi / 15)
    xx, xy = c * q(2, 2).real, -c * q(2, 2).imag
    xz, yz = -c * q(2, 1).real, c * q(2, 1).imag
    M = torch.stack([torch.stack([tr - zz / 2 + xx, xy, xz]), torch.stack([xy, tr - zz / 2 - xx, yz]),
                     torch.stack([xz, yz, tr + zz])])
    th, ph, ps = x["ptg"].unbind(1)
    v = x["beta"][torch.arange(case["n"], device=DEV) // x["period"]]
    # R^T v with R = R_z(phi) R_y(theta) R_z(psi)
    v0, v1 = v[:, 0] * ph.cos() + v[:, 1] * ph.sin(), v[:, 1] * ph.cos() - v[:, 0] * ph.sin()
    v0, v2 = v0 * th.cos() - v[:, 2] * th.sin(), v0 * th.sin() + v[:, 2] * th.cos()
    u = torch.stack([v0 * ps.cos() + v1 * ps.sin(), v1 * ps.cos() - v0 * ps.sin(), v2], 1)
    return x["T0"] * (u @ S + x["q"] * ((u @ M) * u).sum(1))
