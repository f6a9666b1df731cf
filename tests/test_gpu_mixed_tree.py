"""Mixed solves whose products take the treecode (from 4e8 node pairs x columns on with
one domain, 1e9 in a batch) against FP64 solves: one column, odd and even column counts,
a zero column, a batch with domains on both sides of the line, with and without graphs,
under a workspace cap (which keeps to the pair kernels) and again on the same context.

Bar, as for the other mixed solves: 1e-10 relative L-infinity between solutions solved
to 1e-12.
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


def _domain(gk, m1, n):
    cen = [2.4 * ((k % 7) + 1j * (k // 7)) for k in range(m1)]
    return gk.DeviceDomain.from_host(wl.circles_unbounded(n, cen, [1.0 - 0.01 * k for k in range(m1)]))


def _gamma(dom, cols):
    x, y = dom.eta.real, dom.eta.imag
    c = [torch.cos((0.2 + 0.1 * k) * x) + (0.3 + k) * torch.sin(0.15 * y + k) for k in range(cols)]
    return torch.stack(c, 1).contiguous()


def _close(a, b):
    err = float((a - b).abs().max() / b.abs().max())
    print(f"  {err:.2e}", flush=True)
    assert err <= 1e-10


@pytest.mark.parametrize("m1,n,cols,inner_tol", [(10, 2048, 1, 0.0), (11, 2040, 1, 1.0), (9, 1024, 5, 1.0),
                                                 (9, 1026, 6, 1.0), (4, 1024, 25, 1.0)])
def test_one_domain(gk, m1, n, cols, inner_tol):
    print(f"[mixed tree] {m1} x {n}, {cols} columns", flush=True)
    dom = _domain(gk, m1, n)
    gam = _gamma(dom, cols)
    if cols > 2:
        gam[:, 1] = 0.0
    opts = dict(restart=10, maxit=20, tol=1e-12)
    ctx = gk.Context(0)
    try:
        ref, href, _, st = ctx.fbie(dom, gam, **opts)
        assert st == 0
        mixed = dict(prec=gk.MIXED, inner_tol=inner_tol, **opts)
        mu, h, infos, st = ctx.fbie(dom, gam, **mixed)
        assert st == 0
        steps = [i["mixed_steps"] if isinstance(i, dict) else i.mixed_steps for i in infos]
        assert max(steps) > 0
        _close(mu, ref)
        _close(h, href)
        again = ctx.fbie(dom, gam, **mixed)
        assert torch.equal(again[0], mu) and torch.equal(again[1], h)
        ad, _, st = ctx.fbie_ad(dom, gam, **mixed)
        assert st == 0
        _close(ad, ctx.fbie_ad(dom, gam, **opts)[0])
    finally:
        ctx.close()


def test_batch_on_both_sides_of_the_line(gk, monkeypatch):
    shapes, cols = [(5, 256), (18, 1024), (3, 70), (12, 1024), (7, 2048)], [5, 18, 2, 11, 7]
    print("[mixed tree] batch", flush=True)
    doms = [_domain(gk, *s) for s in shapes]
    gams = [_gamma(d, c) for d, c in zip(doms, cols)]
    opts = dict(restart=10, maxit=20, tol=1e-12)
    mixed = dict(prec=gk.MIXED, inner_tol=1.0, **opts)

    def solve(**kw):
        ctx = gk.Context(0)
        try:
            mus, hs, _, st = ctx.fbie_batched(doms, gams, **kw)
            assert st == 0
            return mus + hs
        finally:
            ctx.close()

    ref, got = solve(**opts), solve(**mixed)
    for a, b in zip(got, ref):
        _close(a, b)
    # (the batch's launch shape is tuned by timing, the sums' order with it)
    monkeypatch.setenv("GNK_TUNE", "0")
    got = solve(**mixed)
    monkeypatch.setenv("GNK_GRAPH", "0")
    for a, b in zip(solve(**mixed), got):
        assert torch.equal(a, b)
    monkeypatch.delenv("GNK_GRAPH")
    monkeypatch.setenv("GNK_WORKSPACE_MB", "4096")
    for a, b in zip(solve(**mixed), ref):
        _close(a, b)
