"""Calls on a card with room for the one-sided direct kernels only (GNK_DEVICE_MB lets
allocations fail as there): what these fit still runs, in the first call of a context
and after others, and gives the same results as with all memory."""
import pytest
import torch

pytestmark = pytest.mark.gpu

OVERRIDE = "GNK_CAUCHY_TPT"      # keeps to the one-sided kernels


def _circles(m1, n):
    import workloads as wl
    from paper_1308_5351_amd import gnk
    return gnk.DeviceDomain.from_host(
        wl.circles_unbounded(n, [2.6 * (k % 9) + 2.6j * (k // 9) for k in range(m1)], [1.0] * m1))


def _fits(calls, mib, monkeypatch, one_sided):
    """The calls' results in one context with that much room, or None."""
    from paper_1308_5351_amd import gnk
    if mib:
        monkeypatch.setenv("GNK_DEVICE_MB", str(mib))
    if one_sided:
        monkeypatch.setenv(OVERRIDE, "2")
    ctx = gnk.Context(0)
    try:
        return [c(ctx) for c in calls]
    except gnk.GnkError as e:
        assert e.status == gnk.ERR_OOM
        return None
    finally:
        ctx.close()
        for k in ("GNK_DEVICE_MB", OVERRIDE):
            monkeypatch.delenv(k, raising=False)


def _need(call, monkeypatch):
    """The least room in MiB for a call by the one-sided kernels."""
    lo, hi = 0, 1 << 12
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lo, hi = (lo, mid) if _fits([call], mid, monkeypatch, True) else (mid, hi)
    return hi


@pytest.fixture(scope="module")
def calls():
    from paper_1308_5351_amd import gnk
    gen = torch.Generator().manual_seed(1)
    d, big, odd = _circles(21, 2048), _circles(13, 2048), _circles(20, 1500)
    x = torch.randn(d.N, 2, generator=gen, dtype=torch.float64).cuda()
    xb = torch.randn(big.N, 2, generator=gen, dtype=torch.float64).cuda()
    xo = torch.randn(odd.N, generator=gen, dtype=torch.float64).cuda()
    w = torch.randn(d.N, generator=gen, dtype=torch.complex128).cuda()
    opts = dict(restart=10, maxit=3, tol=1e-11)
    mixed = dict(restart=10, maxit=3, tol=1e-11, prec=gnk.MIXED, inner_tol=1.0)
    return {"fbie": lambda c: c.fbie(d, x[:, 0].contiguous(), **opts)[0],
            "fbie_ad": lambda c: c.fbie_ad(d, x[:, 0].contiguous(), **opts)[0],
            "mixed": lambda c: c.fbie(d, x, **mixed)[0],
            "batch": lambda c: torch.cat(c.fbie_batched([d, big], [x, xb], **mixed)[0]),
            "odd": lambda c: c.fbie(odd, xo, **opts)[0],
            "sum": lambda c: c.cauchy_sum(d.eta, w)}


@pytest.mark.parametrize("name", ["fbie", "fbie_ad", "mixed", "batch", "odd", "sum"])
def test_first_call(calls, name, monkeypatch):
    monkeypatch.setenv("GNK_TUNE", "0")      # one launch shape in all contexts
    call = calls[name]
    need = _need(call, monkeypatch)
    ref = _fits([call], 0, monkeypatch, False)[0]
    got = _fits([call, call], need, monkeypatch, False)
    print(f"[full card] {name}: {need} MiB", flush=True)
    assert got is not None
    for g in got:
        # residuals of 1e-11 on both sides, the systems' condition below 1e2 (the sum: rounding)
        assert float((g - ref).abs().max() / ref.abs().max()) <= 1e-9


@pytest.mark.parametrize("first,then", [("fbie", "mixed"), ("sum", "odd"), ("mixed", "batch"), ("odd", "fbie")])
def test_after_another_call(calls, first, then, monkeypatch):
    """A second call that fits in a context of its own fits after the first."""
    monkeypatch.setenv("GNK_TUNE", "0")
    need = max(_need(calls[first], monkeypatch), _need(calls[then], monkeypatch))
    ref = _fits([calls[then]], 0, monkeypatch, False)[0]
    got = _fits([calls[first], calls[then]], need, monkeypatch, False)
    print(f"[full card] {first}, {then}: {need} MiB", flush=True)
    assert got is not None
    assert float((got[1] - ref).abs().max() / ref.abs().max()) <= 1e-9


def test_too_little_room_is_still_an_error(calls, monkeypatch):
    need = _need(calls["fbie"], monkeypatch)
    assert _fits([calls["fbie"]], need - 1, monkeypatch, False) is None
