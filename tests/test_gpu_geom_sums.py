"""The geometric derivative's sums with one to five groups (pairs of them per launch
plane, the last plane of an odd count alone), at the ends of its tiles of 128 targets
and with source splits that leave a wave without sources: against the oracle's dense
derivative. As for the other geometric gradients 1e-11 of the largest entry: the
terms carry |d|^-2, and N of them meet at 1e-16 each.
"""
import numpy as np
import pytest
import torch

from oracle import gradient as og

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("G", [1, 2, 3, 5])
@pytest.mark.parametrize("m1,n", [(1, 4), (1, 62), (1, 126), (1, 128), (1, 130), (3, 86), (5, 102), (3, 514)])
def test_geom_vjp_groups(m1, n, G):
    from paper_1308_5351_amd import gnk as gk
    print(f"[geom] m1={m1} n={n} G={G}", flush=True)
    rng = np.random.default_rng([m1, n, G])
    N = m1 * n
    t = 2 * np.pi * np.arange(n) / n
    eta = (1.5 * np.arange(m1)[:, None] + 0.5 * np.exp(-1j * t) + 0.05 * np.exp(2j * t)).ravel()
    etap = (0 * np.arange(m1)[:, None] - 0.5j * np.exp(-1j * t) + 0.1j * np.exp(2j * t)).ravel()
    A = 1.0 + 0.3 * (rng.normal(size=N) + 1j * rng.normal(size=N))
    v = [rng.normal(size=N) for _ in range(G)]
    terms = [(("FB", "FC")[k % 2], rng.normal(), rng.normal(size=N), k % G) for k in range(G + 2)]
    ref = og.bilinear_geom_grad(eta, etap, A, n, [(op, c * u, v[g]) for op, c, u, g in terms])
    cuda = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    dom = gk.DeviceDomain(m1, n, cuda(eta), cuda(etap), cuda(A))
    V = [cuda(x) for x in v]
    ctx = gk.Context(0)
    try:
        got = ctx.geom_vjp(dom, [({"FB": gk.OP_FB, "FC": gk.OP_FC}[op], c, cuda(u), V[g]) for op, c, u, g in terms])
        for g, r in zip(got, ref):
            assert np.abs(g.cpu().numpy() - r).max() <= 1e-11 * np.abs(r).max()
    finally:
        ctx.close()
