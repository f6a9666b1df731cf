"""The treecode's order and interaction lists, made on the GPU, at the sizes where
their kernels change: one leaf and less, ragged leaves and blocks, leaf counts and
point counts on both sides of the one-block sort (4096) and of the sort's tiles
(2048), equal points, one cluster, points that are not finite.

Tolerance: far_tol bounds each box's truncation relative to sum |w_j|/|z - eta_j|
over the box, so the tree differs from the direct sum by at most far_tol times
that sum, plus the rounding of the two (256 eps of it).
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
EPS = np.finfo(float).eps


@pytest.fixture(scope="module")
def gk():
    from paper_1308_5351_amd import gnk
    return gnk


def _circles(N, n, seed):
    """N nodes on circles of n nodes, placed in random order on a grid."""
    r = np.random.default_rng(seed)
    m = (N + n - 1) // n
    s = int(np.ceil(np.sqrt(m)))
    place = r.permutation(m)
    k, t = np.arange(N) // n, (np.arange(N) % n) * (2 * np.pi / n)
    eta = (place[k] % s) + 1j * (place[k] // s) + 0.35 * np.exp(-1j * t)
    w = r.standard_normal(N) + 1j * r.standard_normal(N)
    return torch.from_numpy(eta).cuda(), torch.from_numpy(w).cuda()


@pytest.mark.parametrize("far_tol", [1e-13, 1e-4])
@pytest.mark.parametrize("N", [1, 63, 256, 257, 513, 4095, 16385, 70001, 1048576 + 300])
def test_tree_sum_matches_plain_sum(gk, N, far_tol):
    print(f"[tree] N={N} far_tol={far_tol}", flush=True)
    eta, w = _circles(N, 300, N)
    ctx = gk.Context(0)
    try:
        S = ctx.cauchy_sum(eta, w, far_tol=far_tol)
        assert torch.equal(S, ctx.cauchy_sum(eta, w, far_tol=far_tol))
        rows = torch.arange(N) if N <= 5000 else torch.from_numpy(np.random.default_rng(1).integers(0, N, 400))
        for a in range(0, len(rows), 64):
            i = rows[a:a + 64].cuda()
            d = eta[i, None] - eta[None, :]
            q = torch.where(d == 0, 0.0, 1.0 / d)
            ref, size = q @ w, q.abs() @ w.abs()
            assert bool(((S[i] - ref).abs() <= (far_tol + 256 * EPS) * size).all())
    finally:
        ctx.close()


@pytest.mark.parametrize("nz", [1, 64, 129, 2048, 4096, 4097, 6143, 6145, 100003])
def test_points_in_any_number(gk, nz):
    """f = 1/(z - c) + 3 outside 24 circles from the tree and, for the first points, from the direct sums."""
    n, m1 = 512, 24
    eta, _ = _circles(n * m1, n, 7)
    cen = eta.view(m1, n).mean(1, keepdim=True)
    etap = (-1j * (eta.view(m1, n) - cen)).reshape(-1)
    f = 1.0 / (eta - cen[3]) + 3.0
    r = np.random.default_rng(nz)
    z = torch.from_numpy(r.integers(-1, 6, nz) + 0.5 + 1j * (r.integers(-1, 6, nz) + 0.5)
                         + 1e-3 * (r.standard_normal(nz) + 1j * r.standard_normal(nz))).cuda()
    ctx = gk.Context(0)
    try:
        t = ctx.fcau(eta, etap, f, z, m1, n, finf=3.0, far_tol=1e-13)
        # the formula itself is exact here to a few hundred eps (n nodes resolve f to rounding)
        assert float((t - (1.0 / (z - cen[3]) + 3.0)).abs().max()) <= 1e-11
        assert torch.equal(t, ctx.fcau(eta, etap, f, z, m1, n, finf=3.0, far_tol=1e-13))
    finally:
        ctx.close()


@pytest.mark.parametrize("nz", [300, 5000])
def test_equal_and_nonfinite_points(gk, nz):
    """All points equal (every code a tie), and a few that are not finite among ordinary ones: those alone give
    non-finite values."""
    n, m1 = 512, 24
    eta, _ = _circles(n * m1, n, 7)
    cen = eta.view(m1, n).mean(1, keepdim=True)
    etap = (-1j * (eta.view(m1, n) - cen)).reshape(-1)
    f = 1.0 / (eta - cen[3]) + 3.0
    z = torch.full((nz,), 1.5 + 2.5j, dtype=torch.complex128, device="cuda")
    want = 1.0 / (z[0] - cen[3]) + 3.0
    ctx = gk.Context(0)
    try:
        t = ctx.fcau(eta, etap, f, z, m1, n, finf=3.0, far_tol=1e-13)
        assert float((t - want).abs().max()) <= 1e-11
        bad = torch.arange(5, nz, 97, device="cuda")
        z[bad] = complex(float("nan"), 0.0)
        t = ctx.fcau(eta, etap, f, z, m1, n, finf=3.0, far_tol=1e-13)
        ok = torch.ones(nz, dtype=torch.bool, device="cuda")
        ok[bad] = False
        assert float((t[ok] - want).abs().max()) <= 1e-11
        assert bool(torch.isnan(t[bad].real).all())
    finally:
        ctx.close()


@pytest.mark.parametrize("far_tol", [1e-15, 1e-8, 1e-5, 1e-2])
@pytest.mark.parametrize("kind", ["circles", "random"])
def test_expansion_orders(gk, kind, far_tol):
    """Every instance of the moments' and conversions' kernels (p = 48, 21, 13 and 6 terms of a box at most), one
    and three weight columns, tiles small beside their boxes (circles) and as large (random nodes: up to 48 terms of
    a tile's expansion). A box's truncation is at most 7/3 far_tol on its own side and 7/3 far_tol/64 on the tile's."""
    N = 20011
    eta, w = _circles(N, 300, 5)
    if kind == "random":
        r = np.random.default_rng(8)
        eta = torch.from_numpy(r.uniform(-1, 1, N) + 1j * r.uniform(-1, 1, N)).cuda()
    w3 = torch.stack([w, w.conj() * 0.5, w.roll(7)], dim=1)
    ctx = gk.Context(0)
    try:
        S = ctx.cauchy_sum(eta, w, far_tol=far_tol)
        S3 = ctx.cauchy_sum(eta, w3, far_tol=far_tol)
        rows = torch.from_numpy(np.random.default_rng(1).integers(0, N, 512)).cuda()
        d = eta[rows, None] - eta[None, :]
        q = torch.where(d == 0, 0.0, 1.0 / d)
        for got, x in ((S, w), (S3[:, 0], w), (S3[:, 1], w3[:, 1]), (S3[:, 2], w3[:, 2])):
            ref, size = q @ x, q.abs() @ x.abs()
            worst = float(((got[rows] - ref).abs() / size).max())
            print(f"[tree] {kind} far_tol {far_tol:g}: {worst:.2e}", flush=True)
            assert worst <= 2.4 * far_tol + 256 * EPS
    finally:
        ctx.close()
