"""Two-sided one-column sums whose last block has waves without nodes: these hold
zero weights in the place of the last node and may add nothing to the streamed
nodes' sums, however close one of those lies to the last node. Here a node of
another block is 2^-33 away from it, at the same offset from its chunk's centre up
to rounding, so that the expanded distance is exactly zero. Tolerance as in the
tests of the two-sided sums, 256 eps of the sum of the term sizes."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [8193, 8250, 8448, 8705, 10305, 43009, 43500, 44100])
def test_node_beside_the_last_one(N):
    from paper_1308_5351_amd import gnk
    print(f"[idle waves] N={N}", flush=True)
    g = torch.Generator().manual_seed(N)
    eta = 40.0 * torch.complex(torch.rand(N, generator=g, dtype=torch.float64),
                               torch.rand(N, generator=g, dtype=torch.float64)) + (9.0 + 9.0j)
    # chunk 3: inside |x|, |y| <= 1 + 2^-33 with its bounding box centred on 0
    r = 1.0 + 2.0 ** -33
    c = 0.9 * torch.polar(torch.ones(64, dtype=torch.float64), torch.arange(64).double() * (2 * np.pi / 64) + 0.01)
    c[0], c[1], c[2], c[3] = r, -r, 1.0j, -1.0j
    eta[192:256] = c
    eta[N - 1] = 1.0
    w = torch.complex(torch.randn(N, generator=g, dtype=torch.float64), torch.randn(N, generator=g, dtype=torch.float64))
    eta, w = eta.cuda(), w.cuda()
    ctx = gnk.Context(0)
    try:
        S = ctx.cauchy_sum(eta, w)
    finally:
        ctx.close()
    worst = 0.0
    for a in range(0, N, 2048):
        rows = torch.arange(a, min(N, a + 2048), device="cuda")
        d = eta[rows, None] - eta[None, :]
        own = torch.arange(len(rows), device="cuda")
        d[own, rows] = 1.0
        q = 1.0 / d
        q[own, rows] = 0.0
        err = ((S[rows] - q @ w).abs() / (q.abs() @ w.abs())).max()
        assert bool(torch.isfinite(err)), a
        worst = max(worst, float(err))
    print(f"  worst {worst / np.finfo(float).eps:.1f} eps", flush=True)
    assert worst <= 256 * np.finfo(float).eps
