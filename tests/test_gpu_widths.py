"""The FP64 pair kernels at every column-group width (1-8) and every way of
splitting more columns into groups, with one and two targets per lane (the line
lies at 1024 targets for one column, 2048 for several), domains smaller than a
tile, and source splits that do not divide the nodes: against a plain FP64 sum,
for the nodes themselves and for separate points.

Tolerance: as for the two-sided sums, a term carries about ten roundings, amplified
by at most 25 in the far form: |S - S_ref| <= 256 eps sum_j |w_j|/|d_ij|.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
EPS = np.finfo(float).eps


@pytest.fixture(scope="module")
def ctx():
    from paper_1308_5351_amd import gnk
    c = gnk.Context(0)
    yield c
    c.close()


def _circles(m1, n):
    t = torch.arange(n, dtype=torch.float64) * (2 * np.pi / n)
    e = torch.polar(torch.ones(n, dtype=torch.float64), -t)
    k = torch.arange(m1)
    cen = torch.complex((k % 6).double(), torch.div(k, 6, rounding_mode="floor").double())
    return (cen[:, None] + 0.4 * e).reshape(-1).cuda()


def _columns(N, cols, seed):
    g = torch.Generator().manual_seed(seed)
    return torch.complex(torch.randn(N, cols, generator=g, dtype=torch.float64),
                         torch.randn(N, cols, generator=g, dtype=torch.float64)).cuda()


@pytest.mark.parametrize("cols", [1, 2, 3, 4, 5, 6, 7, 8, 9, 11, 13, 17])
@pytest.mark.parametrize("m1,n", [(2, 10), (2, 32), (3, 126), (3, 340), (2, 512), (5, 410), (3, 682), (11, 600)])
def test_sums_of_every_width(ctx, m1, n, cols):
    print(f"[widths] {m1} x {n}, {cols}", flush=True)
    N = m1 * n
    eta, w = _circles(m1, n), _columns(N, cols, N + cols)
    S = ctx.cauchy_sum(eta, w)
    few = torch.empty(cols, N, dtype=w.dtype, device="cuda")   # planned without the extra splits
    wc = w.t().contiguous()
    assert ctx.lib.gnk_cauchy_sum_noalloc(ctx.h, N, eta.data_ptr(), wc.data_ptr(), cols, few.data_ptr()) == 0
    d = eta[:, None] - eta[None, :]
    d.fill_diagonal_(1.0)
    q = 1.0 / d
    q.fill_diagonal_(0.0)
    ref, size = q @ w, q.abs() @ w.abs()
    assert float(((S - ref).abs() / size).max()) <= 256 * EPS
    assert float(((few.t() - ref).abs() / size).max()) <= 256 * EPS


@pytest.mark.parametrize("cols", [1, 2, 3, 4, 5, 6, 7, 8, 10])
@pytest.mark.parametrize("nz", [1, 63, 1023, 1024, 2047, 2050])
def test_interior_values_of_every_width(ctx, nz, cols):
    print(f"[widths] {nz} points, {cols}", flush=True)
    n = 700
    t = torch.arange(n, dtype=torch.float64) * (2 * np.pi / n)
    e = torch.polar(torch.ones(n, dtype=torch.float64), t).cuda()
    g = torch.Generator().manual_seed(nz)
    z = (torch.polar(0.9 * torch.rand(nz, generator=g, dtype=torch.float64).sqrt(),
                     2 * np.pi * torch.rand(nz, generator=g, dtype=torch.float64))).cuda()
    f = _columns(n, cols, nz + cols)
    got = ctx.fcau(e, 1j * e, f, z, 1, n)
    q = (1j * e)[None, :] / (e[None, :] - z[:, None])
    den, size = q.sum(1, keepdim=True), q.abs()
    ref = (q @ f) / den
    bound = 256 * EPS * (size @ f.abs() + ref.abs() * size.sum(1, keepdim=True)) / den.abs()
    assert bool(((got.reshape(nz, cols) - ref).abs() <= bound).all())


@pytest.mark.parametrize("n", [6, 10, 70, 254, 258, 510, 514, 600, 2046, 3838, 3840, 3842, 5000, 7680, 7690])
@pytest.mark.parametrize("cols", [1, 2])
def test_circulant_of_other_lengths(ctx, n, cols):
    """The direct circulant product at the ends of its tiles of 256 outputs and 3840
    inputs, with inputs that do not fill the last four and an odd number of vectors:
    n terms of two roundings each, 1e-13 of the largest sum of their sizes. The
    reference's column takes its arguments on the near side, cot(pi d/n) =
    -cot(pi (n - d)/n): beyond, rounding of pi d/n costs the dense oracle's largest
    entries a relative n eps, 9e-14 of the sum at n = 7690."""
    import workloads as wl
    from paper_1308_5351_amd import gnk
    m1 = 3
    print(f"[circulant] n={n} cols={cols}", flush=True)
    dom = wl.circles_unbounded(n, [0j, 3.0 + 0.5j, -2.5 + 2.0j], [1.0, 0.7, 0.5])
    x = _columns(m1 * n, cols, n).real.contiguous()
    y = ctx.apply(gnk.DeviceDomain.from_host(dom), gnk.OP_LHAT, x).reshape(m1 * n, cols)
    d = np.arange(n)
    near = np.minimum(d, n - d)
    col = np.where(2 * d > n, -1.0, 1.0) * (-1.0) ** d / np.tan(np.pi * np.where(near == 0, 0.5 * n, near) / n) / n
    col[[0, n // 2]] = 0.0
    L = torch.from_numpy(col).cuda()[torch.from_numpy((d[:, None] - d[None, :]) % n).cuda()]
    for k in range(m1):
        blk = slice(k * n, (k + 1) * n)
        err = (y[blk] - L @ x[blk]).abs().max() / (L.abs() @ x[blk].abs()).max()
        assert float(err) < 1e-13, k
