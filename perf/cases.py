"""Workloads of the solver's public entry points, from one small solve to the
largest: what a program that uses this package has it do.

A case is a dict of plain values; ``kind`` names the entry point:

* ``fbie``     one or several right-hand sides of (I - N) mu = -M gamma, with h
               (``Context.fbie``): FP64, mixed precision or the far field by
               expansions (``far_tol``)
* ``fbie_ad``  (I + N* + J) mu = gamma (``Context.fbie_ad``)
* ``batched``  many domains of uneven size with one right-hand side per hole
               (``Context.fbie_batched``)
* ``grad``     a loss on h through Fourier curves and FBIE, forward and backward
               (``autograd.fourier_curve``, ``autograd.fbie``)
* ``fcau``     an analytic function at points of the domain from its boundary
               values (``Context.fcau``), summed directly or with ``far_tol``
* ``slit``     the map onto a slit domain (``Context.slit_map``)

Right-hand sides are gamma = Re[A f] - h_k with f analytic in the domain and
h_k one constant per component, so mu = Im[A f] and h = h_k in closed form.
"""
import math
import random

import numpy as np
import torch

from paper_1308_5351_amd import autograd, gnk

DEV = "cuda"
KMIN, NTERMS = -7, 16   # Fourier terms of a boundary curve


def listed():
    return [
        # the smallest solve: one hole in the unit disc (latency and launches)
        dict(name="fbie_2x256", kind="fbie", bounded=True, m1=2, n=256, cols=1, restart=25, tol=1e-12),
        # the ordinary solve of the method's listing: 16 holes in the unit disc
        dict(name="fbie_17x1024", kind="fbie", bounded=True, m1=17, n=1024, cols=1, restart=25, tol=1e-12),
        # the adjoint equation on a mesh that is no power of two
        dict(name="fbie_ad_17x720", kind="fbie_ad", bounded=True, m1=17, n=720, restart=25, tol=1e-12),
        # several right-hand sides of one domain, ragged: 11 holes, 600 nodes, 5 columns
        dict(name="fbie_11x600_5cols", kind="fbie", bounded=False, m1=11, n=600, cols=5, restart=25, tol=1e-12),
        # the largest direct solve: 129 perturbed circles of 2048 nodes
        dict(name="fbie_129x2048", kind="fbie", bounded=False, m1=129, n=2048, cols=1, restart=60, tol=1e-13),
        # boundaries close to each other, mixed precision: many steps per solve
        dict(name="fbie_close_25x2048_mixed", kind="fbie", bounded=False, m1=25, n=2048, cols=1, restart=256,
             tol=1e-13, gap=0.01, mixed=True),
        # uneven domains with a right-hand side per hole in one mixed batch, refined every 10 steps
        dict(name="batched_8_mixed", kind="batched", ndom=8, m1_max=40, n_max=2048, mix=3, restart=10, tol=1e-12,
             mixed=True),
        # shape gradient of sum_k h_k^2: forward solve, adjoint solve, geometric derivatives
        dict(name="grad_33x1024", kind="grad", m1=33, n=1024, restart=60, tol=1e-13),
        # an analytic function at points of the domain, summed directly
        dict(name="fcau_17x1024_65536", kind="fcau", bounded=True, m1=17, n=1024, nz=65536, far_tol=0.0),
        # the same at many points around a large boundary, with expansions
        dict(name="fcau_289x1024_200003_far", kind="fcau", bounded=False, m1=289, n=1024, nz=200003, far_tol=1e-13),
        # the largest boundary: 1089 curves of 4096 nodes, far field by expansions
        dict(name="fbie_1089x4096_far", kind="fbie", bounded=False, m1=1089, n=4096, cols=1, restart=25, tol=1e-12,
             far_tol=1e-13),
        # conformal map of the exterior of five close circles onto circular slits
        dict(name="slit_5x4096", kind="slit", n=4096, eps=0.01, restart=25, maxit=40, tol=1e-12),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _mesh(rng, lo, hi):
    """Nodes per curve: half of the draws a power of two, the others any even number."""
    if rng.random() < 0.5:
        return 1 << rng.randint((lo - 1).bit_length(), hi.bit_length() - 1)
    return 2 * _log_int(rng, lo // 2, hi // 2)


def draw(rng):
    kind = rng.choice(["fbie", "fbie", "fbie_ad", "cols", "close", "batched", "grad", "fcau", "far", "fcau_far", "slit"])
    if kind == "fbie":
        if rng.random() < 0.5:
            return dict(kind="fbie", bounded=True, m1=rng.randint(2, 17), n=_mesh(rng, 256, 2048), cols=1, restart=25,
                        tol=1e-12)
        return dict(kind="fbie", bounded=False, m1=_log_int(rng, 2, 110), n=_mesh(rng, 256, 2048), cols=1, restart=60,
                    tol=1e-13)
    if kind == "fbie_ad":
        return dict(kind="fbie_ad", bounded=True, m1=rng.randint(2, 17), n=_mesh(rng, 256, 2048), restart=25, tol=1e-12)
    if kind == "cols":
        return dict(kind="fbie", bounded=False, m1=rng.randint(2, 33), n=_mesh(rng, 256, 1024), cols=rng.randint(2, 16),
                    restart=25, tol=1e-12)
    if kind == "close":
        return dict(kind="fbie", bounded=False, m1=rng.randint(4, 25), n=rng.choice([1024, 1536, 2048]), cols=1,
                    restart=256, tol=1e-13, gap=round(rng.uniform(0.01, 0.05), 4), mixed=rng.random() < 0.7)
    if kind == "batched":
        return dict(kind="batched", ndom=rng.randint(2, 8), m1_max=rng.randint(6, 30), n_max=rng.choice([512, 1024, 2048]),
                    mix=rng.randint(0, 999), restart=10, tol=1e-12, mixed=rng.random() < 0.7)
    if kind == "grad":
        return dict(kind="grad", m1=_log_int(rng, 3, 33), n=_mesh(rng, 128, 1024), restart=60, tol=1e-13)
    if kind == "fcau":
        return dict(kind="fcau", bounded=True, m1=rng.randint(2, 17), n=_mesh(rng, 256, 1024),
                    nz=_log_int(rng, 200, 65536), far_tol=0.0)
    if kind == "far":
        return dict(kind="fbie", bounded=False, m1=_log_int(rng, 60, 900), n=_mesh(rng, 512, 4096), cols=1, restart=25,
                    tol=1e-12, far_tol=1e-13)
    if kind == "fcau_far":
        return dict(kind="fcau", bounded=False, m1=_log_int(rng, 60, 500), n=_mesh(rng, 512, 2048),
                    nz=_log_int(rng, 5000, 200003), far_tol=1e-13)
    return dict(kind="slit", n=_mesh(rng, 1024, 4096), eps=round(math.exp(rng.uniform(math.log(0.01), math.log(0.1))), 4),
                restart=25, maxit=40, tol=1e-12)


# ------------------------------------------------------------------ geometry
def _rng(seed, salt):
    return np.random.default_rng([13085351, salt, int(seed)])


def _grid(m1):
    s = int(math.ceil(math.sqrt(m1)))
    i = np.arange(m1)
    return (i % s - 0.5 * (s - 1)) + 1j * (i // s - 0.5 * (s - 1))


def _circles_coef(m1, r):
    """Fourier coefficients of m1 perturbed circles (clockwise), about 1.2 apart."""
    cen = 1.2 * _grid(m1) + r.uniform(-0.08, 0.08, m1) + 1j * r.uniform(-0.08, 0.08, m1)
    rad = r.uniform(0.25, 0.35, m1)
    ks = np.arange(KMIN, KMIN + NTERMS)
    c = (r.uniform(-1, 1, (m1, NTERMS)) + 1j * r.uniform(-1, 1, (m1, NTERMS))) * (0.1 / math.sqrt(2)) * rad[:, None]
    c[:, (ks == 0) | (ks == 1)] = 0
    s = np.sum(np.abs(ks) * np.abs(c), axis=1)
    c *= np.minimum(1.0, 0.5 * rad / s)[:, None]
    c[:, ks == 0] = cen[:, None]
    c[:, ks == 1] = rad[:, None]
    return c, cen, rad


def _curves(coef, ks, n):
    """eta, eta', eta'' of the clockwise curves sum_k c_k e^{-ikt} (torch, complex128)."""
    c = torch.from_numpy(coef).to(DEV)
    k = torch.from_numpy(ks).to(DEV, torch.float64)
    p = torch.arange(n, device=DEV, dtype=torch.float64)
    ph = torch.polar(torch.ones(len(ks), n, device=DEV, dtype=torch.float64),
                     -2 * math.pi * torch.remainder(k[:, None] * p[None, :], n) / n)
    w = [c, c * (-1j * k), c * (-(k * k))]
    return tuple((x.to(torch.complex128) @ ph).reshape(-1) for x in w)


def _bounded(m1, n, r):
    """Unit circle (ccw) and m1 - 1 ellipses (cw), the origin in the domain: eta, eta', eta'', centres, semi-axes."""
    t = 2 * math.pi * np.arange(n) / n
    parts = [(np.exp(1j * t), 1j * np.exp(1j * t), -np.exp(1j * t))]
    holes = []
    while len(holes) < m1 - 1:
        a, b, phi = (r.uniform(0.2, 0.3), r.uniform(0.1, 0.2), r.uniform(0, np.pi)) if m1 == 2 else \
            (r.uniform(0.03, 0.08), r.uniform(0.03, 0.08), r.uniform(0, np.pi))
        R = max(a, b)
        c = (0.96 - R) * math.sqrt(r.uniform()) * np.exp(1j * r.uniform(0, 2 * np.pi))
        if abs(c) < R + 0.04 or any(abs(c - h[0]) < R + max(h[1], h[2]) + 0.04 for h in holes):
            continue
        holes.append((c, a, b, phi))
        e = np.exp(1j * phi)
        parts.append((c + e * (a * np.cos(t) - 1j * b * np.sin(t)), e * (-a * np.sin(t) - 1j * b * np.cos(t)),
                      e * (-a * np.cos(t) + 1j * b * np.sin(t))))
    eta, etap, etapp = (torch.from_numpy(np.concatenate([p[q] for p in parts])).to(DEV) for q in range(3))
    return eta, etap, etapp, holes


def _domain(case, seed, salt=1):
    """DeviceDomain of the case, poles in its holes (numpy), and what the points of the domain need."""
    m1, n = case["m1"], case["n"]
    r = _rng(seed, salt)
    if case.get("bounded", False):
        eta, etap, etapp, holes = _bounded(m1, n, r)
        dom = gnk.DeviceDomain(m1, n, eta, etap, eta.clone(), etapp, etap.clone(), 1)
        return dom, np.array([h[0] for h in holes]), holes
    if case.get("gap"):
        # circles that almost touch their neighbours on a square grid
        rad = 0.5 - 0.5 * case["gap"] * r.uniform(0.5, 1.0, m1)
        cen = _grid(m1)
        coef, ks = np.stack([cen, rad.astype(complex)], axis=1), np.array([0, 1])
    else:
        coef, cen, rad = _circles_coef(m1, r)
        ks = np.arange(KMIN, KMIN + NTERMS)
    eta, etap, etapp = _curves(coef, ks, n)
    one = torch.ones_like(eta)
    return gnk.DeviceDomain(m1, n, eta, etap, one, etapp, torch.zeros_like(eta), -1), cen, (cen, rad)


def _poles(poles, r, bounded):
    """Residues, the entire part's factor and the constants h_k of one analytic function."""
    res = (r.uniform(-1, 1, len(poles)) + 1j * r.uniform(-1, 1, len(poles))) * (0.05 if bounded else 0.1)
    return res, (0.5 if bounded else 0.0)


def _f(z, poles, res, entire):
    """sum_k res_k / (z - poles_k) + entire e^z for a torch tensor z."""
    v = entire * torch.exp(z) if entire else torch.zeros_like(z)
    if len(poles) <= 64:
        for p, a in zip(poles, res):
            v = v + complex(a) / (z - complex(p))
        return v
    # many holes: sixteen of them carry a pole
    for q in range(0, len(poles), max(1, len(poles) // 16)):
        v = v + complex(res[q]) / (z - complex(poles[q]))
    return v


def _rhs(dom, poles, seed, cols, bounded):
    """gamma = Re[A f] - h_k, mu = Im[A f], h (all N x cols)."""
    r = _rng(seed, 2)
    g, m, h = [], [], []
    for _ in range(cols):
        res, entire = _poles(poles, r, bounded)
        v = dom.A * _f(dom.eta, poles, res, entire)
        hk = torch.from_numpy(r.uniform(-0.5, 0.5, dom.m1)).to(DEV).repeat_interleave(dom.n)
        g.append(v.real - hk)
        m.append(v.imag)
        h.append(hk)
    if cols == 1:
        return g[0].contiguous(), m[0], h[0]
    return tuple(torch.stack(x, dim=1) for x in (g, m, h))


def _points(case, seed, dom, extra):
    """nz points of the domain in random order, a quarter of them 1e-4..1e-2 from a boundary."""
    nz, r = case["nz"], _rng(seed, 4)
    near = nz // 4
    eta = dom.eta.cpu().numpy()
    if case["bounded"]:
        holes = extra

        def inside(z):
            ok = np.abs(z) < 1.0
            for c, a, b, phi in holes:
                w = (z - c) * np.exp(-1j * phi)
                ok &= (w.real / a) ** 2 + (w.imag / b) ** 2 > 1.0
            return z[ok]

        j = r.integers(0, eta.shape[0], 2 * near + 16)
        d = np.exp(r.uniform(math.log(1e-4), math.log(1e-2), j.shape[0]))
        cen = np.concatenate([[0j], [h[0] for h in holes]])[j // dom.n]
        zn = inside(cen + (eta[j] - cen) * np.where(j < dom.n, 1.0 - d, 1.0 + d))[:near]
        zf = inside(np.sqrt(r.uniform(0, 1, 2 * nz)) * np.exp(2j * np.pi * r.uniform(0, 1, 2 * nz)))[:nz - len(zn)]
    else:
        cen, rad = extra
        j = r.integers(0, eta.shape[0], near)
        d = np.exp(r.uniform(math.log(1e-4), math.log(1e-2), near))
        c = cen[j // dom.n]
        zn = c + (eta[j] - c) * (1.0 + d)
        s = int(math.ceil(math.sqrt(dom.m1)))
        half = 0.6 * s + 1.0
        z = r.uniform(-half, half, 2 * nz) + 1j * r.uniform(-half, half, 2 * nz)
        q = np.clip(np.rint(z.real / 1.2 + 0.5 * (s - 1)), 0, s - 1) + \
            s * np.clip(np.rint(z.imag / 1.2 + 0.5 * (s - 1)), 0, s - 1)
        q = np.minimum(q.astype(int), dom.m1 - 1)
        zf = z[np.abs(z - cen[q]) > 1.5 * rad[q]][:nz - near]
    z = np.concatenate([zn, zf])
    return torch.from_numpy(z[r.permutation(len(z))]).to(DEV)


def _batch_sizes(case):
    """(m1, n) of the domains of a batch: a fixed mix, whatever the seed."""
    q = random.Random(case["mix"])
    return [(q.randint(2, case["m1_max"]), q.choice([x for x in (256, 512, 1024, 2048) if x <= case["n_max"]]))
            for _ in range(case["ndom"])]


def _slit_domain(case, seed):
    r = _rng(seed, 5)
    cen = np.array([0, 1 + 1j, -1 + 1j, -1 - 1j, 1 - 1j])
    eps = case["eps"] * r.uniform(0.9, 1.1)
    rad = np.array([math.sqrt(2) - 1 - eps / 2] + [1 - eps / 2] * 4)
    turn = np.exp(1j * r.uniform(0, 2 * np.pi))
    coef = np.stack([cen * turn, rad * turn], axis=1)
    eta, etap, _ = _curves(coef, np.array([0, 1]), case["n"])
    return eta, etap, complex(2.5j * turn)


# ------------------------------------------------------------------ the cases
def _solver_opts(case):
    o = dict(restart=case["restart"], maxit=case.get("maxit", 20), tol=case["tol"])
    if case.get("mixed"):
        o["prec"] = gnk.MIXED
    return o


def prepare(case, seed):
    ctx = autograd.default_context(torch.cuda.current_device())
    s = dict(case=case, ctx=ctx)
    kind = case["kind"]
    if kind in ("fbie", "fbie_ad"):
        dom, poles, _ = _domain(case, seed)
        s["dom"] = dom
        s["gam"] = _rhs(dom, poles, seed, case.get("cols", 1), case["bounded"])[0]
    elif kind == "batched":
        s["doms"], s["gams"] = [], []
        for d, (m1, n) in enumerate(_batch_sizes(case)):
            dom, poles, _ = _domain(dict(m1=m1, n=n), seed, 10 + d)
            s["doms"].append(dom)
            s["gams"].append(_rhs(dom, poles, 100 * seed + d, m1, False)[0])
    elif kind == "grad":
        coef, _, _ = _circles_coef(case["m1"], _rng(seed, 1))
        s["coef"] = torch.from_numpy(coef).to(DEV)
        eta, _, _ = _curves(coef, np.arange(KMIN, KMIN + NTERMS), case["n"])
        s["gam"] = (eta * eta).real.contiguous()
    elif kind == "fcau":
        dom, poles, extra = _domain(case, seed)
        res, entire = _poles(poles, _rng(seed, 2), case["bounded"])
        s["dom"], s["finf"] = dom, None if case["bounded"] else 3.0
        s["f"] = _f(dom.eta, poles, res, entire) + (0.0 if case["bounded"] else 3.0)
        s["z"] = _points(case, seed, dom, extra)
    else:
        s["eta"], s["etap"], s["alpha"] = _slit_domain(case, seed)
    return s


def run(s):
    case, ctx = s["case"], s["ctx"]
    kind = case["kind"]
    if kind == "fbie":
        mu, h, _, _ = ctx.fbie(s["dom"], s["gam"], far_tol=case.get("far_tol", 0.0), **_solver_opts(case))
        return dict(mu=mu, h=h)
    if kind == "fbie_ad":
        return dict(mu=ctx.fbie_ad(s["dom"], s["gam"], **_solver_opts(case))[0])
    if kind == "batched":
        o = _solver_opts(case)
        if case.get("mixed"):
            o["inner_tol"] = 1.0   # every Arnoldi product mixed, refined at each restart
        mus, hs, _, _ = ctx.fbie_batched(s["doms"], s["gams"], **o)
        return dict(mu=mus, h=hs)
    if kind == "grad":
        coef = s["coef"].detach().requires_grad_(True)
        gam = s["gam"].detach().requires_grad_(True)
        m1, n = case["m1"], case["n"]
        eta, etap, _ = autograd.fourier_curve(coef, KMIN, n, context=ctx)
        mu, h = autograd.fbie(eta, etap, torch.ones_like(eta), gam, m1, n, context=ctx, **_solver_opts(case))
        loss = (h.view(m1, n).mean(1) ** 2).sum()
        loss.backward()
        return dict(mu=mu.detach(), h=h.detach(), g_coef=coef.grad, g_gam=gam.grad)
    if kind == "fcau":
        d = s["dom"]
        return ctx.fcau(d.eta, d.etap, s["f"], s["z"], d.m1, d.n, finf=s["finf"], far_tol=case["far_tol"])
    f, level, _, _ = ctx.slit_map(s["eta"], s["etap"], 5, case["n"], s["alpha"], [0.5 * math.pi] * 5, bounded=False,
                                  **_solver_opts(case))
    return dict(f=f, level=level)


def work(case):
    """One pass: the arrays of the domain and the right-hand sides read once and the results written once; 16
    flops for each pair of nodes and the first column of a product (8 for each further one), with the steps that
    the solve takes; with far_tol, the near field (three leaves of 256 nodes per target) and 8 flops for each of
    20 terms of 30 boxes per target."""
    kind = case["kind"]
    if kind == "batched":
        sizes = [(m1 * n, m1) for m1, n in _batch_sizes(case)]
        steps = 24 if case.get("mixed") else 19
        return dict(bytes=sum(N * (48 + 24 * c) for N, c in sizes), flops=sum(steps * N * N * (8.0 + 8 * c) for N, c in sizes))
    if kind == "slit":
        N = 5 * case["n"]
        return dict(bytes=48 * N, flops=70 * 16.0 * N * N)
    N = case["m1"] * case["n"]
    if kind == "fcau":
        per = (3 * 256 * 24.0 + 30 * 20 * 16.0) if case["far_tol"] else 24.0 * N
        return dict(bytes=48 * N + 32 * case["nz"], flops=per * case["nz"])
    if kind == "grad":
        return dict(bytes=48 * N + 16 * 2 * case["m1"] * NTERMS + 32 * N, flops=(2 * 20 * 16.0 + 64) * N * N)
    cols = case.get("cols", 1)
    steps = 110 if case.get("gap") else 20
    per = (3 * 256 * 16.0 + 30 * 20 * 8.0) if case.get("far_tol") else N * (8.0 + 8 * cols)
    return dict(bytes=N * ((80 if kind == "fbie_ad" else 48) + 24 * cols), flops=steps * per * N)


# ----------------------------------------------------- the same in plain torch
def _kernel(eta, etap, A, n):
    """K_ij = (2/n) (A_i / A_j) eta'_j / (eta_j - eta_i), 0 on the diagonal; N is its imaginary part, M its real part."""
    d = eta[None, :] - eta[:, None]
    d = d + torch.eye(eta.shape[0], device=eta.device, dtype=d.dtype)
    K = (2.0 / n) * A[:, None] * (etap / A)[None, :] / d
    return K - torch.diag(torch.diagonal(K))


def _exact_fbie_ad(case, seed):
    if case["m1"] * case["n"] > 20000:
        return None
    dom, poles, _ = _domain(case, seed)
    gam = _rhs(dom, poles, seed, 1, case["bounded"])[0]
    n = dom.n
    B = _kernel(dom.eta, dom.etap, dom.A, n).imag
    d = dom.eta[:, None] - dom.eta[None, :]
    d.fill_diagonal_(1.0)
    E = dom.etap[None, :] / d
    E.fill_diagonal_(0.0)
    e = 1 - dom.c - (2.0 / n) * E.sum(1).imag + (2.0 / n) * (dom.etapp / dom.etap - dom.Ap / dom.A).imag
    del d, E
    M = B.t().contiguous()
    del B
    M.view(dom.m1, n, dom.m1, n).diagonal(dim1=0, dim2=2).add_(1.0 / n)
    M += torch.diag(e)
    return dict(mu=torch.linalg.solve(M, gam[:, None])[:, 0])


def _exact_grad(case, seed):
    m1, n = case["m1"], case["n"]
    N = m1 * n
    if N > 6000:
        return None
    coef = torch.from_numpy(_circles_coef(m1, _rng(seed, 1))[0]).to(DEV)
    ks = np.arange(KMIN, KMIN + NTERMS)
    eta0 = _curves(coef.cpu().numpy(), ks, n)[0]
    gam = (eta0 * eta0).real.contiguous().requires_grad_(True)
    coef.requires_grad_(True)
    k = torch.from_numpy(ks).to(DEV, torch.float64)
    p = torch.arange(n, device=DEV, dtype=torch.float64)
    ph = torch.polar(torch.ones(NTERMS, n, device=DEV, dtype=torch.float64),
                     -2 * math.pi * torch.remainder(k[:, None] * p[None, :], n) / n)
    eta, etap = (coef @ ph).reshape(-1), ((coef * (-1j * k)) @ ph).reshape(-1)
    K = _kernel(eta, etap, torch.ones_like(eta), n)
    q = torch.arange(n, device=DEV)
    dd = q[:, None] - q[None, :]
    L = torch.where(dd == 0, 0.0, (1.0 - 2.0 * (dd % 2)) / n / torch.tan(math.pi * dd.to(torch.float64).where(dd != 0, 0.5) / n))
    Aop = 2 * torch.eye(N, device=DEV, dtype=torch.float64) + torch.diag(K.imag.sum(1)) - K.imag
    Cop = K.real - torch.diag(K.real.sum(1)) + torch.block_diag(*[L] * m1)
    mu = torch.linalg.solve(Aop, -(Cop @ gam)[:, None])[:, 0]
    h = 0.5 * (Cop @ mu - Aop @ gam)
    (h.view(m1, n).mean(1) ** 2).sum().backward()
    return dict(mu=mu.detach(), h=h.detach(), g_coef=coef.grad, g_gam=gam.grad)


def exact(case, seed):
    kind = case["kind"]
    if kind == "fbie":
        dom, poles, _ = _domain(case, seed)
        _, mu, h = _rhs(dom, poles, seed, case.get("cols", 1), case["bounded"])
        return dict(mu=mu, h=h)
    if kind == "fbie_ad":
        return _exact_fbie_ad(case, seed)
    if kind == "batched":
        mus, hs = [], []
        for d, (m1, n) in enumerate(_batch_sizes(case)):
            dom, poles, _ = _domain(dict(m1=m1, n=n), seed, 10 + d)
            _, mu, h = _rhs(dom, poles, 100 * seed + d, m1, False)
            mus.append(mu)
            hs.append(h)
        return dict(mu=mus, h=hs)
    if kind == "grad":
        return _exact_grad(case, seed)
    if kind == "fcau":
        dom, poles, extra = _domain(case, seed)
        res, entire = _poles(poles, _rng(seed, 2), case["bounded"])
        return _f(_points(case, seed, dom, extra), poles, res, entire) + (0.0 if case["bounded"] else 3.0)
    return None
