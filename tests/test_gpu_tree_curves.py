"""The treecode's leaves and tiles end with their curve: curves of a leaf's nodes, of a
few more, of a tile and a remainder, and (below 64 nodes, where leaves run across
curves) shorter; one, two and three columns; interior points; and a mixed solve with
such curves. Solves and values with far_tol 1e-13 against the direct sums.

Bar: 1e-10 relative L-infinity, as for the other solves (tol 1e-12), and for values
1e-11: far_tol of the sum of term sizes, amplified by the ratio's denominator.
"""
import numpy as np
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gk():
    from paper_1308_5351_amd import gnk
    return gnk


@pytest.fixture(scope="module")
def ctx(gk):
    c = gk.Context(0)
    yield c
    c.close()


def _domain(gk, m1, n):
    cen = [2.6 * ((k % 6) + 1j * (k // 6)) for k in range(m1)]
    return gk.DeviceDomain.from_host(wl.circles_unbounded(n, cen, [1.0 - 0.01 * (k % 9) for k in range(m1)]))


def _gamma(dom, cols):
    x, y = dom.eta.real, dom.eta.imag
    return torch.stack([torch.cos((0.2 + 0.1 * k) * x) + torch.sin(0.15 * y + k) for k in range(cols)], 1).contiguous()


def _close(a, b, tol):
    err = float((a - b).abs().max() / b.abs().max())
    print(f"  {err:.2e}", flush=True)
    assert err <= tol


@pytest.mark.parametrize("cols", [1, 2, 3])
@pytest.mark.parametrize("m1,n", [(30, 50), (30, 62), (30, 64), (30, 66), (30, 100), (20, 126), (20, 128), (20, 130),
                                  (12, 190), (12, 258), (9, 600)])
def test_solves(gk, ctx, m1, n, cols):
    print(f"[curves] {m1} x {n}, {cols}", flush=True)
    dom = _domain(gk, m1, n)
    gam = _gamma(dom, cols)
    mu, h, _, st = ctx.fbie(dom, gam, tol=1e-12, far_tol=1e-13)
    ref, href, _, st2 = ctx.fbie(dom, gam, tol=1e-12)
    assert st == 0 and st2 == 0
    _close(mu, ref, 1e-10)
    _close(h, href, 1e-10)


@pytest.mark.parametrize("m1,n", [(30, 62), (30, 66), (20, 130), (9, 600)])
def test_values_at_points(gk, ctx, m1, n):
    print(f"[curves] values, {m1} x {n}", flush=True)
    dom = _domain(gk, m1, n)
    f = 1.0 / (dom.eta - (0.1 + 0.05j)) + 0.5 / (dom.eta - 2.6)
    g = torch.Generator().manual_seed(n)
    t = torch.rand(3001, generator=g, dtype=torch.float64).cuda()
    z = 1.3 + 1.3j + 0.25 * torch.polar(t, 40 * t) + 2.6 * torch.floor(4 * t)
    a = ctx.fcau(dom.eta, dom.etap, f, z, m1, n, finf=0.0, far_tol=1e-13)
    _close(a, ctx.fcau(dom.eta, dom.etap, f, z, m1, n, finf=0.0), 1e-11)


def test_mixed_solve(gk, ctx):
    print("[curves] mixed", flush=True)
    dom = _domain(gk, 34, 606)
    gam = _gamma(dom, 3)
    opts = dict(restart=10, maxit=20, tol=1e-12)
    mu, h, _, st = ctx.fbie(dom, gam, prec=gk.MIXED, inner_tol=1.0, **opts)
    ref, href, _, st2 = ctx.fbie(dom, gam, **opts)
    assert st == 0 and st2 == 0
    _close(mu, ref, 1e-10)
    _close(h, href, 1e-10)
