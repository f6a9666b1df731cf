"""The Cauchy integral at points some of which are nodes, with two targets per lane
(from 2048 points on) and every column-group width: those take the node's value, and
every other point, the lane's second target 64 places away among them, the plain
FP64 sum's, within 256 eps of the sum of the term sizes."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
EPS = np.finfo(float).eps


@pytest.mark.parametrize("cols", [1, 2, 3, 4, 5, 6, 7, 8, 9])
@pytest.mark.parametrize("far_tol", [0.0, 1e-12])
def test_points_beside_points_on_nodes(cols, far_tol):
    from paper_1308_5351_amd import gnk
    print(f"[point on node] {cols} columns, far_tol {far_tol}", flush=True)
    n, nz = 700, 4100
    t = torch.arange(n, dtype=torch.float64) * (2 * np.pi / n)
    e = torch.polar(torch.ones(n, dtype=torch.float64), t)
    g = torch.Generator().manual_seed(cols)
    z = torch.polar(0.9 * torch.rand(nz, generator=g, dtype=torch.float64).sqrt(),
                    2 * np.pi * torch.rand(nz, generator=g, dtype=torch.float64))
    at = torch.tensor([5, 70, 1000, 2047, 2048, 3333, 4099])      # both targets of a lane, the last point
    node = torch.tensor([0, 3, 698, 64, 128, 350, 699])
    z[at] = e[node]
    e, z = e.cuda(), z.cuda()
    f = torch.complex(torch.randn(n, cols, generator=g, dtype=torch.float64),
                      torch.randn(n, cols, generator=g, dtype=torch.float64)).cuda()
    ctx = gnk.Context(0)
    try:
        got = ctx.fcau(e, 1j * e, f, z, 1, n, far_tol=far_tol).reshape(nz, cols)
    finally:
        ctx.close()
    assert torch.equal(got[at.cuda()], f[node.cuda()])
    rest = torch.ones(nz, dtype=torch.bool)
    rest[at] = False
    rest = rest.cuda()
    q = (1j * e)[None, :] / (e[None, :] - z[rest][:, None])
    den, size = q.sum(1, keepdim=True), q.abs()
    ref = (q @ f) / den
    bound = (256 * EPS if far_tol == 0.0 else 1e-11) * (size @ f.abs() + ref.abs() * size.sum(1, keepdim=True)) / den.abs()
    assert bool(((got[rest] - ref).abs() <= bound).all())
