"""The two-sided one-column Cauchy sums against a plain FP64 sum, at the sizes
where their blocks, wave tiles and chunks end: one column from 8000 nodes on
(blocks of 1024 nodes, 256 per wave; from 40000 on blocks of 2048), even and odd
block counts, a last block with one node, with empty waves and with a ragged
chunk. The one-sided kernel on the same input (gnk_cauchy_sum_noalloc) as well.

Tolerance: a far pair's distance and difference of sums amplify rounding by at
most 25 (separation 1.5 (r_t + r_s)), with about ten roundings per pair, so each
term is within 256 eps of its size: |S - S_ref| <= 256 eps sum_j |w_j|/|d_ij|.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gk():
    from paper_1308_5351_amd import gnk
    return gnk


def _nodes(N, kind, seed):
    g = torch.Generator().manual_seed(seed)
    if kind == "random":      # no chunk is far
        eta = torch.complex(torch.rand(N, generator=g, dtype=torch.float64), torch.rand(N, generator=g, dtype=torch.float64))
    else:                     # circles of 500 nodes: far and near chunks, chunks on two circles
        k = torch.arange(N) // 500
        t = (torch.arange(N) % 500).double() * (2 * np.pi / 500)
        eta = torch.complex((k % 9).double(), (k // 9).double()) + 0.4 * torch.polar(torch.ones_like(t), -t)
    w = torch.complex(torch.randn(N, generator=g, dtype=torch.float64), torch.randn(N, generator=g, dtype=torch.float64))
    return eta.cuda(), w.cuda()


def _reference(eta, w, rows):
    d = eta[rows, None] - eta[None, :]
    r = torch.arange(len(rows), device=d.device)
    d[r, rows] = 1.0
    q = 1.0 / d
    q[r, rows] = 0.0
    return q @ w, q.abs() @ w.abs()


@pytest.mark.parametrize("kind", ["random", "circles"])
@pytest.mark.parametrize("N", [8000, 8192, 8193, 9216, 9279, 10305, 12240, 16640, 39999, 40000, 40961, 43008, 45120])
def test_two_sided_sum_matches_plain_sum(gk, N, kind):
    print(f"[sym] N={N} {kind}", flush=True)
    eta, w = _nodes(N, kind, N)
    ctx = gk.Context(0)
    try:
        S = ctx.cauchy_sum(eta, w)
        assert torch.equal(S, ctx.cauchy_sum(eta, w))
        one = torch.empty_like(w)
        st = ctx.lib.gnk_cauchy_sum_noalloc(ctx.h, N, eta.data_ptr(), w.data_ptr(), 1, one.data_ptr())
        assert st == 0
        worst = 0.0
        for a in range(0, N, 2048):
            rows = torch.arange(a, min(N, a + 2048), device="cuda")
            ref, size = _reference(eta, w, rows)
            for X in (S, one):
                worst = max(worst, float(((X[rows] - ref).abs() / size).max()))
        print(f"  worst {worst / np.finfo(float).eps:.1f} eps", flush=True)
        assert worst <= 256 * np.finfo(float).eps
    finally:
        ctx.close()


@pytest.mark.parametrize("n", [1364, 1024])
def test_operators_of_one_and_two_columns_agree(gk, n):
    """Every operator (with its diagonal from a leading column) applied to one column (two-sided sums) and to the
    same column twice (one-sided sums of two columns)."""
    import workloads as wl
    dom, gam = wl.config1(n=n, m_inner=8)
    dd = gk.DeviceDomain.from_host(dom)
    x = torch.from_numpy(gam[:, 0]).cuda()
    ctx = gk.Context(0)
    try:
        for op in (gk.OP_FB, gk.OP_FC, gk.OP_GB, gk.OP_FB_T, gk.OP_FC_T, gk.OP_GB_T, gk.OP_FB_U, gk.OP_GB_U):
            print(f"[sym] operator {op}", flush=True)
            y1 = ctx.apply(dd, op, x)
            y2 = ctx.apply(dd, op, torch.stack([x, x], dim=1))
            # sums of about 1e4 terms with 256 eps each of their size, against results of their order
            assert float((y1 - y2[:, 0]).abs().max() / y2.abs().max()) <= 1e-11
    finally:
        ctx.close()


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_solves_of_one_and_three_columns_agree(gk, prec):
    """One column (two-sided FP64 products, in the mixed solve beside one-sided mixed ones) against three."""
    import workloads as wl
    dom, gam = wl.config1(n=1000, m_inner=8)
    dd = gk.DeviceDomain.from_host(dom)
    x = torch.from_numpy(gam[:, 0]).cuda()
    ctx = gk.Context(0)
    kw = dict(restart=30, tol=1e-13, prec=gk.MIXED if prec == "mixed" else gk.FP64)
    try:
        mu1, h1, _, s1 = ctx.fbie(dd, x, **kw)
        mu3, h3, _, s3 = ctx.fbie(dd, torch.stack([x, 2 * x, -x], dim=1), **kw)
        assert s1 == 0 and s3 == 0
        for a, b in ((mu1, mu3[:, 0]), (h1, h3[:, 0]), (2 * mu1, mu3[:, 1])):
            # both solutions have a residual of 1e-13; the system's condition is below 1e2
            assert float((a - b).abs().max() / x.abs().max()) <= 1e-10
    finally:
        ctx.close()


@pytest.mark.parametrize("m1,n", [(6, 1364), (9, 1024), (17, 1024)])
def test_mixed_product_of_one_column(gk, m1, n):
    """A mixed product of one column, at sizes whose FP64 products are two-sided: it
    takes the node records, not the compact weights. 1e-5 as for the other mixed
    products (FP32 far tiles, about 1e-7)."""
    import workloads as wl
    print(f"[sym] mixed {m1} x {n}", flush=True)
    dom = gk.DeviceDomain.from_host(wl.circles_unbounded(n, [2.6 * (k % 5) + 2.6j * (k // 5) for k in range(m1)], [1.0] * m1))
    g = torch.Generator().manual_seed(n)
    x = torch.randn(dom.N, 2, generator=g, dtype=torch.float64).cuda()
    for op in (gk.OP_FB, gk.OP_FB_T):
        ctx = gk.Context(0)
        try:
            y = ctx.apply(dom, op, x[:, 0].contiguous(), prec=gk.MIXED)   # the context's first product
            two = ctx.apply(dom, op, x)
            again = ctx.apply(dom, op, x[:, 0].contiguous(), prec=gk.MIXED)
            for v in (y, again):
                assert float((v - two[:, 0]).abs().max() / two[:, 0].abs().max()) < 1e-5
        finally:
            ctx.close()
