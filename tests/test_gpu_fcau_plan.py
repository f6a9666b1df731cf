"""The Cauchy integral of few nodes (below 128, where a launch plan has one source
split at most) at numbers of points around one round of the card's wave slots:
64-node circles at grids of points, directly and by the treecode, against a plain
FP64 sum. Tolerance: a term carries about ten roundings, 256 eps of the sum of the
term sizes; the treecode at 1e-12 within 1e-11.
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


@pytest.mark.parametrize("far_tol", [0.0, 1e-12])
@pytest.mark.parametrize("n,cols,nz", [(64, 1, 196608), (64, 1, 196609), (64, 1, 262144), (64, 1, 294785),
                                       (100, 2, 131073), (100, 2, 150000), (126, 2, 196481), (64, 4, 163857),
                                       (64, 7, 150000), (3, 1, 262144), (128, 1, 262144)])
def test_few_nodes_at_many_points(ctx, n, cols, nz, far_tol):
    print(f"[fcau plan] {n} nodes, {cols} columns, {nz} points, far_tol {far_tol}", flush=True)
    t = torch.arange(n, dtype=torch.float64) * (2 * np.pi / n)
    e = torch.polar(torch.ones(n, dtype=torch.float64), t).cuda()
    g = torch.Generator().manual_seed(nz + cols)
    z = torch.polar(0.9 * torch.rand(nz, generator=g, dtype=torch.float64).sqrt(),
                    2 * np.pi * torch.rand(nz, generator=g, dtype=torch.float64)).cuda()
    f = torch.complex(torch.randn(n, cols, generator=g, dtype=torch.float64),
                      torch.randn(n, cols, generator=g, dtype=torch.float64)).cuda()
    got = ctx.fcau(e, 1j * e, f, z, 1, n, far_tol=far_tol)
    q = (1j * e)[None, :] / (e[None, :] - z[:, None])
    den, size = q.sum(1, keepdim=True), q.abs()
    ref = (q @ f) / den
    bound = (256 * EPS if far_tol == 0.0 else 1e-11) * (size @ f.abs() + ref.abs() * size.sum(1, keepdim=True)) / den.abs()
    assert bool(((got.reshape(nz, cols) - ref).abs() <= bound).all())
