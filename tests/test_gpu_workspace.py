"""Device memory that a context holds after a call: what the call's own kernels need,
not the partial sums of kernels that it does not run."""
import gc

import pytest
import torch

pytestmark = pytest.mark.gpu


def _circles(m1, n):
    import workloads as wl
    from paper_1308_5351_amd import gnk
    return gnk.DeviceDomain.from_host(
        wl.circles_unbounded(n, [2.6 * (k % 9) + 2.6j * (k // 9) for k in range(m1)], [1.0] * m1))


def _held(call, monkeypatch, **env):
    """Bytes that a new context's call leaves allocated outside torch."""
    from paper_1308_5351_amd import gnk
    for k, v in env.items():
        monkeypatch.setenv(k, v)
    try:
        gc.collect()
        ctx = gnk.Context(0)
        call(ctx)          # torch's own buffers and the library's host-mapped ones
        ctx.close()
        torch.cuda.synchronize()
        ctx = gnk.Context(0)
        free = torch.cuda.mem_get_info()[0]
        call(ctx)
        torch.cuda.synchronize()
        held = free - torch.cuda.mem_get_info()[0]
        ctx.close()
        return held
    finally:
        for k in env:
            monkeypatch.delenv(k)


def test_calls_without_direct_sums(monkeypatch):
    """Treecode solves and sums, Cauchy integrals and geometric derivatives of 130 x 2048
    nodes. Per node: the restart's basis (8 (restart + 1)) and about 120 of further vectors,
    the node records (16 per field and column), splits of 16 per column, and lists and
    expansions of about 100; the direct sums' partial ones would take 2100 more."""
    from paper_1308_5351_amd import gnk
    d = _circles(130, 2048)
    x = torch.randn(d.N, dtype=torch.float64, device="cuda")
    w = torch.randn(d.N, dtype=torch.complex128, device="cuda")
    z = 100.0 + torch.randn(1000, dtype=torch.complex128, device="cuda")
    for name, per_node, call in (
            ("far", 1000, lambda c: c.fbie(d, x, restart=10, maxit=1, far_tol=1e-10)),
            ("far ad", 1000, lambda c: c.fbie_ad(d, x, restart=10, maxit=1, far_tol=1e-10)),
            ("sum tree", 800, lambda c: c.cauchy_sum(d.eta, w, far_tol=1e-10)),
            ("fcau tree", 800, lambda c: c.fcau(d.eta, d.etap, w, z, d.m1, d.n, finf=0.0, far_tol=1e-10)),
            ("fcau", 800, lambda c: c.fcau(d.eta, d.etap, w, z, d.m1, d.n, finf=0.0)),
            ("geom", 1000, lambda c: c.geom_vjp(d, [(gnk.OP_FB, 1.0, x, x)]))):
        held = _held(call, monkeypatch)
        print(f"[workspace] {name}: {held / d.N:.0f} bytes per node", flush=True)
        assert held <= per_node * d.N, name


@pytest.mark.parametrize("m1,n", [(17, 1024), (36, 2048)])
def test_products_of_several_columns(m1, n, monkeypatch):
    """Two columns run one-sided kernels only: they hold no more than where those alone
    are allowed (16 MB for the runtime's rounding)."""
    d = _circles(m1, n)
    w = torch.randn(d.N, 2, dtype=torch.complex128, device="cuda")
    g = torch.randn(d.N, 2, dtype=torch.float64, device="cuda")
    for call in (lambda c: c.cauchy_sum(d.eta, w), lambda c: c.fbie(d, g, restart=10, maxit=1)):
        held, one = _held(call, monkeypatch), _held(call, monkeypatch, GNK_CAUCHY_TPT="2")
        print(f"[workspace] {m1} x {n}: {held >> 20} MiB, one-sided {one >> 20}", flush=True)
        assert held <= one + (16 << 20)
