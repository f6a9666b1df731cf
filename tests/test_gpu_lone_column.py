"""Columns over full groups of eight at the sizes from which they go alone (one from
5000 targets, two over one group from 32000 nodes on), for the nodes and for separate points, whose one-column
groups take the far form. Tolerance as in the tests of the other widths: 256 eps of
the sum of the term sizes."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
EPS = np.finfo(float).eps


def _columns(N, cols, seed):
    g = torch.Generator().manual_seed(seed)
    return torch.complex(torch.randn(N, cols, generator=g, dtype=torch.float64),
                         torch.randn(N, cols, generator=g, dtype=torch.float64)).cuda()


@pytest.fixture(scope="module")
def ctx():
    from paper_1308_5351_amd import gnk
    c = gnk.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("N,cols", [(4998, 9), (4998, 17), (5000, 8), (5000, 9), (5000, 10), (5000, 17), (5130, 9),
                                    (31990, 10), (32000, 10), (32000, 18)])
def test_sums(ctx, N, cols):
    print(f"[lone column] {N}, {cols}", flush=True)
    t = torch.arange(N, dtype=torch.float64) * (2 * np.pi / 500)
    k = torch.arange(N) // 500
    eta = (torch.complex((k % 8).double(), (k // 8).double()) + 0.4 * torch.polar(torch.ones_like(t), -t)).cuda()
    w = _columns(N, cols, N + cols)
    S = ctx.cauchy_sum(eta, w)
    for a in range(0, N, 5000):
        rows = torch.arange(a, min(N, a + 5000), device="cuda")
        own = torch.arange(len(rows), device="cuda")
        d = eta[rows, None] - eta[None, :]
        d[own, rows] = 1.0
        q = 1.0 / d
        q[own, rows] = 0.0
        assert float(((S[rows] - q @ w).abs() / (q.abs() @ w.abs())).max()) <= 256 * EPS


@pytest.mark.parametrize("nrhs", [7, 8, 9, 16])
@pytest.mark.parametrize("nz", [4999, 5000, 5100])
def test_interior_values(ctx, nz, nrhs):
    print(f"[lone column] {nz} points, {nrhs}", flush=True)
    n = 1000
    t = torch.arange(n, dtype=torch.float64) * (2 * np.pi / n)
    e = torch.polar(torch.ones_like(t), t)
    s = torch.arange(nz, dtype=torch.float64)      # along a spiral: near and far tiles
    z = torch.polar(0.05 + 0.9 * s / nz, s * (8 * np.pi / nz))
    z[[70, nz - 1]] = e[[5, 700]]
    e, z, f = e.cuda(), z.cuda(), _columns(n, nrhs, nz + nrhs)
    got = ctx.fcau(e, 1j * e, f, z, 1, n)
    assert torch.equal(got[[70, nz - 1]], f[[5, 700]])
    rest = torch.ones(nz, dtype=torch.bool)
    rest[[70, nz - 1]] = False
    rest = rest.cuda()
    q = (1j * e)[None, :] / (e[None, :] - z[rest][:, None])
    den, size = q.sum(1, keepdim=True), q.abs()
    ref = (q @ f) / den
    bound = 256 * EPS * (size @ f.abs() + ref.abs() * size.sum(1, keepdim=True)) / den.abs()
    assert bool(((got[rest] - ref).abs() <= bound).all())
