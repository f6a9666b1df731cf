"""The Gram-Schmidt kernels at the ends of their tilings: columns shorter than a
wave, chunks of every fill (the last block of two entries, one wave's worth, a full
block), 8 / 16 and more basis vectors (the register and the two-pass updates, groups
of eight and their remainders), several columns of unequal domains in one batch (blocks
past the end of the short ones), and so many blocks that their partial sums are added
up by a launch of their own. The solutions meet the residual asked for, and the
Arnoldi relation holds: the estimate that the Hessenberg column carries agrees with
the true residual of the next cycle's start.

The estimate's tolerance: b - A x comes with rounding of about N^(1/2) eps |A| |x|,
1e-13 of |b| here, and CGS2 keeps the basis orthogonal to rounding, so estimate and
true residual agree to 1e-12 of |b|.
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


def _domain(gk, m1, n, gap=0.12):
    cen = [(2.0 + gap) * ((k % 40) + 1j * (k // 40)) for k in range(m1)]
    return gk.DeviceDomain.from_host(wl.circles_unbounded(n, cen, [1.0] * m1))


def _gamma(N, cols, seed):
    g = torch.Generator().manual_seed(seed)
    return torch.randn(N, cols, generator=g, dtype=torch.float64).cuda()


def _agree(infos, tol):
    for i in infos:
        i = i if isinstance(i, dict) else i.as_dict()
        print(f"  {i['inner_it']} steps, {i['outer_it']} cycles, {i['relres']:.2e} {i['true_relres']:.2e}", flush=True)
        assert i["flag"] == 0 and i["true_relres"] <= tol
        assert abs(i["relres"] - i["true_relres"]) <= 1e-12


@pytest.mark.parametrize("restart", [2, 3, 8, 9, 16, 17, 25, 48])
@pytest.mark.parametrize("m1,n", [(1, 10), (2, 66), (3, 86), (2, 130), (5, 206), (7, 300), (6, 514)])
def test_solves_at_tiling_edges(gk, ctx, m1, n, restart):
    print(f"[gs] {m1} x {n}, restart {restart}", flush=True)
    dom = _domain(gk, m1, n)
    mu, infos, st = ctx.fbie_ad(dom, _gamma(dom.N, 2, dom.N + restart), restart=restart, maxit=300, tol=1e-9)
    assert st == 0
    _agree(infos, 1e-9)


def test_unequal_domains_and_columns(gk, ctx):
    shapes, cols = [(1, 10), (9, 400), (2, 66), (4, 258)], [3, 1, 2, 5]
    doms = [_domain(gk, *s) for s in shapes]
    gams = [_gamma(d.N, c, d.N) for d, c in zip(doms, cols)]
    print("[gs] batch", flush=True)
    mus, _, infos, st = ctx.fbie_batched(doms, gams, restart=30, maxit=60, tol=1e-9)
    assert st == 0
    for d, g, mu, inf in zip(doms, gams, mus, infos):
        _agree(inf, 1e-9)
        one, _, _, _ = ctx.fbie(d, g, restart=30, maxit=60, tol=1e-12)
        # the batch's residual of 1e-9 |b| against a system of condition below 1e3
        assert float((mu - one).abs().max() / one.abs().max()) <= 1e-6


def test_partial_sums_of_many_blocks(gk, ctx):
    """1069056 nodes: 522 blocks of 2048, the sums of their partials in a launch of
    their own; the products by the treecode (far_tol 1e-13)."""
    dom = _domain(gk, 261, 4096, gap=0.6)
    gam = _gamma(dom.N, 1, 5)
    print("[gs] 261 x 4096", flush=True)
    mu, infos, st = ctx.fbie_ad(dom, gam, restart=25, tol=1e-9, far_tol=1e-13)
    assert st == 0
    _agree(infos, 1e-9)
