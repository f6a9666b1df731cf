"""The geometric derivative, whose kernel shares a reciprocal between a lane's two
targets: two nodes in one place make their own gradients non-finite and nobody
else's, and domains of any scale give the scaled gradients."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,twins", [(300, (7, 40)), (300, (7, 200)), (300, (70, 299)), (1000, (100, 900))])
@pytest.mark.parametrize("G", [1, 2, 3])
def test_geometric_derivative_beside_coincident_nodes(N, twins, G):
    """Node i's gradient with respect to A takes sums at i alone: at the other nodes it
    equals that of the plain sums (1e-11, as the other geometric gradients)."""
    from paper_1308_5351_amd import gnk
    print(f"[coincident] geom N={N} {twins} G={G}", flush=True)
    rng = np.random.default_rng([N, G])
    t = 2 * np.pi * np.arange(N) / N
    eta = np.exp(1j * t) + 0.2 * np.exp(-2j * t)
    etap = 1j * np.exp(1j * t) - 0.4j * np.exp(-2j * t)
    eta[twins[1]] = eta[twins[0]]
    A = 1.0 + 0.3 * (rng.normal(size=N) + 1j * rng.normal(size=N))
    v = [rng.normal(size=N) for _ in range(G)]
    u = [rng.normal(size=N) for _ in range(G)]
    cuda = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    dom = gnk.DeviceDomain(1, N, cuda(eta), cuda(etap), cuda(A))
    ctx = gnk.Context(0)
    try:
        got = ctx.geom_vjp(dom, [((gnk.OP_FB, gnk.OP_FC)[k % 2], 1.0, cuda(u[k]), cuda(v[k])) for k in range(G)])
    finally:
        ctx.close()
    with np.errstate(all="ignore"):
        d = eta[:, None] - eta[None, :]
        np.fill_diagonal(d, 1.0)
        q = 1.0 / d
    np.fill_diagonal(q, 0.0)
    rest = np.setdiff1d(np.arange(N), twins)
    b, kap = etap / A, 2.0 / N
    R1 = R2 = T1 = T2 = 0.0
    for k in range(G):
        z = 1j if k % 2 == 0 else 1.0
        e = v[k][:, None] - v[k][None, :]
        qr, er = q[rest], e[rest]
        R1 = R1 + kap * A[rest] * z * u[k][rest] * ((er * qr) @ b)
        R2 = R2 - kap * A[rest] * z * u[k][rest] * ((er * qr ** 2) @ b)
        T1 = T1 + (er * qr) @ (A * z * u[k])
        T2 = T2 + (er * qr ** 2) @ (A * z * u[k])
    ref = [np.conj(R2 - kap * b[rest] * T2), np.conj(kap * T1 / A[rest]), np.conj((R1 - kap * b[rest] * T1) / A[rest])]
    for x, r in zip(got, ref):
        x = x.cpu().numpy()
        assert np.abs(x[rest] - r).max() <= 1e-11 * np.abs(r).max()
        assert not np.isfinite(x[list(twins)]).any()


@pytest.mark.parametrize("scale", [1e-90, 1e90])
def test_geometric_derivative_of_scaled_domain(scale):
    """The operators do not change when eta and eta' are scaled together: the gradients
    with respect to those scale by 1/scale, that of A not at all, also where the product
    of two squared distances is out of range. 1e-11, as the other geometric gradients."""
    from paper_1308_5351_amd import gnk
    print(f"[coincident] geom scale={scale}", flush=True)
    N = 600
    rng = np.random.default_rng(5)
    t = 2 * np.pi * np.arange(N) / N
    eta = np.exp(1j * t) + 0.2 * np.exp(-2j * t)
    etap = 1j * np.exp(1j * t) - 0.4j * np.exp(-2j * t)
    A = 1.0 + 0.3 * (rng.normal(size=N) + 1j * rng.normal(size=N))
    cuda = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    terms = [(op, 1.0, cuda(rng.normal(size=N)), cuda(rng.normal(size=N))) for op in (gnk.OP_FB, gnk.OP_FC)]
    ctx = gnk.Context(0)
    try:
        ref = ctx.geom_vjp(gnk.DeviceDomain(1, N, cuda(eta), cuda(etap), cuda(A)), terms)
        got = ctx.geom_vjp(gnk.DeviceDomain(1, N, cuda(scale * eta), cuda(scale * etap), cuda(A)), terms)
    finally:
        ctx.close()
    for x, r, s in zip(got, ref, (scale, scale, 1.0)):
        # (torch's abs of a complex number squares its parts)
        x = torch.view_as_real(x) * s
        r = torch.view_as_real(r)
        assert float((x - r).abs().max()) <= 1e-11 * float(r.abs().max())
