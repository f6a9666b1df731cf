"""Two nodes in one place make their own Cauchy sums non-finite and nobody else's, at
every width of the pair kernels (one and two targets per lane, two-sided sums with
four and eight nodes per lane), which share a reciprocal among several nodes of a
lane. The other nodes' sums against a plain FP64 sum, 256 eps of the sum of the term
sizes."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
EPS = np.finfo(float).eps


def _check(eta, w, S, twins):
    N = len(eta)
    for a in range(0, N, 2048):
        rows = torch.arange(a, min(N, a + 2048), device="cuda")
        d = eta[rows, None] - eta[None, :]
        own = torch.arange(len(rows), device="cuda")
        d[own, rows] = 1.0
        q = 1.0 / d
        q[own, rows] = 0.0
        other = torch.ones(len(rows), dtype=torch.bool, device="cuda")
        for i in twins:
            if a <= i < a + len(rows):
                other[i - a] = False
        q = q[other]
        err = (S[rows[other]] - q @ w).abs() / (q.abs() @ w.abs())
        assert bool((err <= 256 * EPS).all()), (a, rows[other][~(err <= 256 * EPS).all(-1)][:8])
    for i in twins:
        assert not bool(torch.isfinite(torch.view_as_real(S[i])).any(-1).any())


# twins in one wave's tile, in neighbouring tiles, in different blocks; the last node
@pytest.mark.parametrize("N,twins", [(900, (100, 103)), (900, (10, 899)), (3000, (100, 230)), (3000, (5, 2999)),
                                     (9000, (70, 75)), (9000, (70, 300)), (9000, (70, 800)), (9000, (70, 8000)),
                                     (9000, (70, 8999)), (17000, (64, 9000)), (41000, (70, 75)), (41000, (600, 1200)),
                                     (41000, (600, 30000)), (41000, (3, 40999))])
@pytest.mark.parametrize("cols", [1, 2, 3, 4, 5, 6, 7, 8])
def test_sums_beside_coincident_nodes(N, twins, cols):
    from paper_1308_5351_amd import gnk
    print(f"[coincident] N={N} {twins} cols={cols}", flush=True)
    g = torch.Generator().manual_seed(N + cols)
    rnd = lambda *s: torch.complex(torch.randn(*s, generator=g, dtype=torch.float64),
                                   torch.randn(*s, generator=g, dtype=torch.float64))
    t = torch.arange(N).double() * (2 * np.pi / 500)
    eta = torch.complex((torch.arange(N) // 500 % 9).double(), (torch.arange(N) // 4500).double()) \
        + 0.4 * torch.polar(torch.ones(N, dtype=torch.float64), -t)
    eta[twins[1]] = eta[twins[0]]
    eta, w = eta.cuda(), rnd(N, cols).cuda()
    ctx = gnk.Context(0)
    try:
        S = ctx.cauchy_sum(eta, w)
    finally:
        ctx.close()
    _check(eta, w, S.reshape(N, cols), twins)
