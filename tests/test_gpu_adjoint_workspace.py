"""Workspace of the FP64 adjoint: graphs that hold its addresses, several passes, no memory.

The adjoint's binned and per-sample forms sum the same products in different orders (and the
atomics in any order): at most a few hundred additions of relative error 2^-53 each, so 1e-12
of the largest value bounds the difference of two of its results.
"""
import os
import subprocess
import sys

import numpy as np
import pytest
import torch

import workloads as W
from paper_2201_03478_amd import api

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
L, K = 24, 3


def _inputs(n, seed=5):
    a, b = (torch.from_numpy(v).cuda() for v in (W.sky_alm(L, 1), W.beam_alm(L, K, 2, kind="flat")))
    p = torch.from_numpy(W.uniform_pointings(n, seed)).cuda()
    return a, b, p, torch.from_numpy(np.random.default_rng(seed).standard_normal(n)).cuda()


def _close(x, y):
    return float((x - y).abs().max()) <= 1e-12 * float(y.abs().max())


def _captured(stream, call):
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=stream):
        call()
    return g


@pytest.mark.parametrize("n", [3000, 20_000])
def test_adjoint_captured_above_the_workspace_it_has(n):
    """A captured adjoint with more samples than any call before it, replayed between eager
    adjoints that grow the workspace."""
    a, b, p, y = _inputs(n)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        plan = api.Plan(L, K, "fp64")
        out = plan.adjoint(b, p[:2900].clone(), y[:2900].clone())
        g = _captured(s, lambda: plan.adjoint(b, p, y, out=out))
        ref = api.Plan(L, K, "fp64").adjoint(b, p, y)
        for m in (200, 5000, 50_000):
            out.zero_()
            g.replay()
            torch.cuda.synchronize()
            assert _close(out, ref), m
            _, _, q, z = _inputs(m, 6)
            eager = plan.adjoint(b, q, z)
            assert _close(eager, api.Plan(L, K, "fp64").adjoint(b, q, z))
        torch.cuda.synchronize()


def test_adjoint_graph_outlives_growth():
    """A binned adjoint captured within its workspace stays valid when later calls outgrow it."""
    a, b, p, y = _inputs(20_000)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        plan = api.Plan(L, K, "fp64")
        out = plan.adjoint(b, p, y)
        ref = out.clone()
        g = _captured(s, lambda: plan.adjoint(b, p, y, out=out))
        for m in (30_000, 90_000, 250_000):
            _, _, q, z = _inputs(m, 7)
            plan.adjoint(b, q, z)
            junk = torch.full((4_000_000,), -1, dtype=torch.int64, device="cuda")
            out.zero_()
            g.replay()
            torch.cuda.synchronize()
            assert _close(out, ref), m
            del junk


def test_interpolation_graph_survives_a_larger_adjoint():
    """The adjoint leaves the interpolation's workspace (which a graph may hold) as it is."""
    a, b, p, _ = _inputs(6000)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        plan = api.Plan(L, K, "fp64")
        plan.set_sky_beam(a, b)
        tod = plan.interpolate(p)
        ref = tod.clone()
        g = _captured(s, lambda: plan.interpolate(p, out=tod))
        for m in (5000, 100_000):
            order = plan.debug_stage(2, 6000)
            _, _, q, z = _inputs(m, 8)
            plan.adjoint(b, q, z)
            assert torch.equal(plan.debug_stage(2, 6000), order)
            tod.zero_()
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(tod, ref)


@pytest.mark.parametrize("limit,n,passes", [(3000, 3000, 1), (3000, 3001, 2), (3000, 9000, 3), (9000, 27_001, 4)])
def test_adjoint_in_several_passes(monkeypatch, limit, n, passes):
    """Passes of up to 3000 samples (one workgroup bins them) and of 9000 (the general path)."""
    a, b, p, y = _inputs(n)
    one = api.Plan(L, K, "fp64")
    monkeypatch.setenv("SC_BIN_PASS_MAX", str(limit))
    several = api.Plan(L, K, "fp64")
    monkeypatch.delenv("SC_BIN_PASS_MAX")
    several.enable_timing(True)
    got = several.adjoint(b, p, y)
    assert several.stage_times()["binning"][1] == passes
    assert _close(got, one.adjoint(b, p, y))
    assert _close(several.adjoint_beam(a, p, y), one.adjoint_beam(a, p, y))


CHILD = """
import sys
sys.path[:0] = [%r, %r]
import test_gpu_adjoint_workspace as t
a, b, p, y = t._inputs(9000)
plan = t.api.Plan(t.L, t.K, "fp64")
plan.set_sky_beam(a, b)
t.np.save(sys.argv[1], plan.adjoint(b, p, y).cpu().numpy())
try:
    plan.interpolate(p)
    raise SystemExit("no allocation failed")
except t.api.N.ScError as e:
    assert "hipMallocAsync" in str(e), e
print("CHILD_OK")
"""


def test_adjoint_without_memory_for_its_workspace(tmp_path):
    """With every allocation after the plan's 16 and the adjoint's 2 refused, the adjoint
    scatters sample by sample; an interpolation then reports the missing memory."""
    f = str(tmp_path / "grad.npy")
    r = subprocess.run([sys.executable, "-c", CHILD % (ROOT, os.path.join(ROOT, "tests")), f], capture_output=True,
                       text=True, timeout=110, env=dict(os.environ, SC_FAIL_ALLOC_AFTER="18"))
    assert r.returncode == 0 and "CHILD_OK" in r.stdout, r.stdout + r.stderr
    _, b, p, y = _inputs(9000)
    assert _close(torch.from_numpy(np.load(f)).cuda(), api.Plan(L, K, "fp64").adjoint(b, p, y))
