"""Performance cases of the distillation low-mode-averaging path.

Each case is one pass through the entry points of paper_2201_09729_amd.dlma as a
user's program calls them, over the lattices, batch sizes, precisions and options of
this repository's workloads (4^4 to 24^3 x 48; one to 128 right-hand sides; FP64 and
FP32, FP16, BF16 storage; forward, adjoint and backward).  Inputs are drawn on the GPU
from a seed: links U = exp(i eps H) (eps = 0.25), spin-diluted smooth orthonormal
timeslice modes and Z2 wall noise as sources, decaying Gaussian fields as solutions.
`exact` restates every result in plain complex128 torch.
"""
import math

import torch

from paper_2201_09729_amd import dlma

DEV = "cuda"
EPS, CSW = 0.25, 1.2
C128 = torch.complex128


def listed():
    return [
        # D on one point source of the smallest lattice (4^4): a check or a toy run, all latency
        {"name": "operator_4_n1", "kind": "operator", "lat": "4x4x4x4", "rhs": 1, "dagger": False},
        # D^dag on the 12 columns of a point propagator at the headline lattice
        {"name": "operator_dag_24x48_n12", "kind": "operator", "lat": "48x24x24x24", "rhs": 12, "dagger": True},
        # a new configuration of an ensemble: load links, build the clover term, apply D to a field
        {"name": "configuration_24x48", "kind": "configuration", "lat": "48x24x24x24", "rhs": 1},
        # the plain FP64 solve of one source, 8^3 x 16
        {"name": "solve_fp64_8x16_n1", "kind": "solve", "lats": "16x8x8x8:m0:n0:p1", "prec": "fp64", "kappa": 0.120},
        # a differentiable FP32-storage solve and its backward (adjoint solve), ragged lattice and batch
        {"name": "gradient_fp32_ragged_n11", "kind": "gradient", "lat": "18x10x6x14", "rhs": 11, "prec": "mix_fp32",
         "kappa": 0.120},
        # one perambulator: 32 modes x 4 spins on 16^3 x 32 in one FP16 multi-RHS solve
        {"name": "solve_fp16_16x32_n128", "kind": "solve", "lats": "32x16x16x16:m32:n0:p0", "prec": "mix_fp16",
         "kappa": 0.121},
        # distillation and stochastic sources together at the headline lattice (the largest)
        {"name": "solve_fp16_24x48_n96", "kind": "solve", "lats": "48x24x24x24:m16:n4:p0", "prec": "mix_fp16",
         "kappa": 0.121},
        # several configurations of uneven volume in one BF16 solve
        {"name": "solve_bf16_uneven_n160", "kind": "solve",
         "lats": "24x12x12x12:m12:n6:p0 24x12x12x12:m8:n0:p0 32x16x16x16:m4:n2:p0", "prec": "mix_bf16", "kappa": 0.120},
        # Laplacian modes of every timeslice
        {"name": "modes_16x32_n32", "kind": "modes", "lat": "32x16x16x16", "nev": 32, "nt": 32, "tol": 1e-12, "block": 0},
        # (1 - box) on the wall sources of 8 noise vectors at the headline lattice
        {"name": "project_24x48_n32", "kind": "project", "lat": "48x24x24x24", "nev": 32, "rhs": 32, "mode": 1},
        # all correlator pieces of one configuration: 32 modes, 128 distillation and 2 x 16 noise solutions
        {"name": "correlators_16x32", "kind": "correlators", "lat": "32x16x16x16", "nev": 32, "dist": 32, "noise": 4,
         "ndil": 1, "backward": False},
        # correlators and their gradient with respect to every solution; odd counts, colour dilution
        {"name": "correlators_grad_12x24", "kind": "correlators", "lat": "24x12x12x12", "nev": 21, "dist": 13, "noise": 6,
         "ndil": 3, "backward": True},
    ]


def draw(rng):
    """One more case of the same ranges: extents even (the library's rule), counts odd and even."""
    def size(lo, hi):  # spread over the logarithm
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    def lattice(limit):
        while True:
            s = size(2, 12)  # spatial half extent
            d = [2 * max(1, s + rng.choice((-1, 0, 0, 0, 1))) for _ in range(3)]
            t = 2 * size(2, 24)
            if t * d[0] * d[1] * d[2] <= limit:
                return "%dx%dx%dx%d" % (t, *d)

    kind = rng.choice(("operator", "configuration", "solve", "solve", "solve", "gradient", "modes", "project", "correlators"))
    if kind in ("operator", "configuration"):
        lat = lattice(663552)
        n = min(size(1, 24), max(1, 10_000_000 // _volume(lat)))
        c = {"kind": kind, "lat": lat, "rhs": n}
        if kind == "operator":
            c["dagger"] = rng.random() < 0.5
        return c
    if kind == "solve":
        prec = rng.choice(("fp64", "mix_fp32", "mix_fp16", "mix_fp16", "mix_bf16"))
        budget = {"fp64": 6_000_000, "mix_fp32": 10_000_000, "mix_fp16": 24_000_000, "mix_bf16": 12_000_000}[prec]
        parts = []
        for _ in range(rng.choice((1, 1, 1, 2, 3))):
            lat = lattice(663552 if not parts else 60000)
            m, nn, p = rng.choice(((size(1, 32), 0, 0), (size(1, 16), size(1, 4), 0), (0, 0, size(1, 12)), (0, size(1, 8), 0)))
            while (4 * m + 8 * nn + p) * _volume(lat) > budget and 4 * m + 8 * nn + p > 1:
                m, nn, p = m // 2, nn // 2, max(p // 2, 0 if m // 2 + nn // 2 else 1)
            parts.append("%s:m%d:n%d:p%d" % (lat, m, nn, p))
        return {"kind": "solve", "lats": " ".join(parts), "prec": prec, "kappa": rng.choice((0.119, 0.120, 0.121))}
    if kind == "gradient":
        lat = lattice(150000)
        n = min(size(1, 24), max(1, 3_000_000 // _volume(lat)))
        return {"kind": kind, "lat": lat, "rhs": n, "prec": rng.choice(("fp64", "mix_fp32", "mix_fp16")),
                "kappa": rng.choice((0.119, 0.120, 0.121))}
    if kind == "modes":
        while True:
            lat = lattice(200000)
            t, z, y, x = _dims(lat)
            if 3 * z * y * x >= 192:
                break
        nev = min(size(2, 40), 3 * z * y * x // 24)
        return {"kind": kind, "lat": lat, "nev": nev, "nt": rng.choice((1, t // 2, t)), "tol": 1e-12,
                "block": rng.choice((0, 0, nev + max(8, nev // 2)))}
    if kind == "project":
        lat = lattice(663552)
        n = min(size(1, 64), max(1, 24_000_000 // _volume(lat)))
        nev = min(size(1, 64), 3 * _volume(lat) // _dims(lat)[0])
        return {"kind": kind, "lat": lat, "nev": nev, "rhs": n, "mode": rng.choice((0, 1))}
    lat = lattice(150000)
    v = _volume(lat)
    nev = min(size(1, 48), 3 * v // _dims(lat)[0])
    ndil = rng.choice((1, 1, 2, 3, 6))
    nd = min(size(1, 48), nev, max(1, 4_000_000 // v))
    nn = max(1, min(size(1, 8), 1_000_000 // v))
    nn = max(1, nn // ndil) * ndil
    return {"kind": "correlators", "lat": lat, "nev": nev, "dist": nd, "noise": nn, "ndil": ndil,
            "backward": rng.random() < 0.5}


# ---------------------------------------------------------------- inputs

def _dims(lat):
    return tuple(int(v) for v in lat.split("x"))


def _volume(lat):
    return math.prod(_dims(lat))


def _parts(case):
    """[(dims, modes, noise vectors, point sources)] of a solve."""
    out = []
    for p in case["lats"].split():
        lat, m, n, q = p.split(":")
        out.append((_dims(lat), int(m[1:]), int(n[1:]), int(q[1:])))
    return out


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _gauss(shape, g):
    return torch.view_as_complex(torch.randn(tuple(shape) + (2,), generator=g, device=DEV, dtype=torch.float64))


def _mul(a, b):
    """3x3 matrix products over leading dimensions."""
    return sum(a[..., :, k, None] * b[..., None, k, :] for k in range(3))


def _links(dims, g):
    a = _gauss(tuple(dims) + (4, 3, 3), g)
    h = 0.5 * (a + a.mH)
    h = h - (torch.diagonal(h, dim1=-2, dim2=-1).sum(-1) / 3)[..., None, None] * torch.eye(3, device=DEV, dtype=C128)
    h = h * (0.25j * EPS)  # exp(i eps H) = (exp(i eps H / 4))^4
    e = torch.eye(3, device=DEV, dtype=C128).expand(h.shape) + h / 14
    for k in range(13, 0, -1):
        e = torch.eye(3, device=DEV, dtype=C128) + _mul(h, e) / k
    e = _mul(e, e)
    return _mul(e, e).contiguous()


def _laplacian(u, v):
    """The covariant Laplacian of timeslices: u [t, z, y, x, 4, 3, 3], v [t, k, z, y, x, 3]."""
    out = -6 * v
    for mu, axis in ((1, 4), (2, 3), (3, 2)):
        um = u[..., mu, :, :][:, None]
        f = torch.roll(v, -1, axis)
        out = out + sum(um[..., :, b] * f[..., b, None] for b in range(3))
        out = out + torch.roll(sum(um[..., b, :].conj() * v[..., b, None] for b in range(3)), 1, axis)
    return out


def _orthonormal(v):
    """Orthonormal vectors v[t, :]: Cholesky QR, twice."""
    s = v.shape
    m = v.reshape(s[0], s[1], -1)
    for _ in range(2):
        gram = (m.conj() @ m.transpose(-1, -2).contiguous())
        low = torch.linalg.cholesky(0.5 * (gram + gram.mH))
        m = torch.linalg.inv(low.conj()) @ m
    return m.reshape(s)


def _modes(u, nev, g):
    """Orthonormal smooth vectors on each timeslice: damped high modes of Gaussian vectors."""
    v = _gauss((u.shape[0], nev) + tuple(u.shape[1:4]) + (3,), g)
    for _ in range(12):
        v = v + _laplacian(u, v) / 12
    return _orthonormal(v).contiguous()


def _sources(dims, m, nn, pts, u, g):
    """Spin-diluted modes and Z2 wall noise with its (1 - box) part on timeslice 0, point sources."""
    t, z, y, x = dims
    b = torch.zeros((4 * m + 8 * nn + pts,) + tuple(dims) + (4, 3), dtype=C128, device=DEV)
    v = _modes(u[:1], max(m, 1), g)[0]
    flat = v.flatten(1)
    xi = (2.0 * torch.randint(0, 2, (nn, z, y, x, 3), generator=g, device=DEV) - 1).to(C128)
    rest = (xi.flatten(1) - (xi.flatten(1) @ flat.conj().T.contiguous()) @ flat).reshape(xi.shape)
    for s in range(4):
        if m:
            b[s:4 * m:4, 0, ..., s, :] = v
        if nn:
            b[4 * m + s:4 * (m + nn):4, 0, ..., s, :] = xi
            b[4 * (m + nn) + s:4 * (m + 2 * nn):4, 0, ..., s, :] = rest
    at = torch.randint(0, math.prod(dims), (1,), generator=g, device=DEV)
    for p in range(pts):
        b[4 * m + 8 * nn + p].view(-1, 12)[at, p % 12] = 1.0
    return b


def prepare(case, seed):
    g = _gen(seed)
    k = case["kind"]
    if k == "solve":
        us = [_links(d, g) for d, *_ in _parts(case)]
        return {"case": case, "us": us,
                "handles": [dlma.dlma_load_gauge(u, case["kappa"], CSW) for u in us],
                "bs": [_sources(*p, u, g) for p, u in zip(_parts(case), us)],
                "opts": dlma.default_opts(prec=case["prec"])}
    dims = _dims(case["lat"])
    u = _links(dims, g)
    st = {"case": case, "u": u}
    if k in ("operator", "configuration"):
        st["x"] = _gauss((case["rhs"],) + dims + (4, 3), g)
        if k == "operator":
            st["g"] = dlma.dlma_load_gauge(u, 0.121, CSW)
        return st
    st["g"] = dlma.dlma_load_gauge(u, case.get("kappa", 0.121), CSW)
    if k == "gradient":
        st["b"] = _gauss((case["rhs"],) + dims + (4, 3), g).requires_grad_()
        # the gradient of a loss like |x|^2: no cancellation in d/dm0
        st["w"] = (st["b"].detach() + 0.3 * _gauss(st["b"].shape, g)).contiguous()
        st["m0"] = torch.tensor(1 / (2 * case["kappa"]) - 4, dtype=torch.float64, requires_grad=True)
        st["opts"] = dlma.default_opts(prec=case["prec"])
    elif k == "modes":
        st["v0"] = _gauss((case["nt"],) + dims[1:] + (3,), g)
    elif k == "project":
        st["v"] = _modes(u[:1], case["nev"], g)[0]
        nn = case["rhs"]
        st["x"] = torch.zeros((nn,) + dims + (4, 3), dtype=C128, device=DEV)
        xi = (2.0 * torch.randint(0, 2, (nn,) + dims[1:] + (3,), generator=g, device=DEV) - 1).to(C128)
        for r in range(nn):
            st["x"][r, 0, ..., r % 4, :] = xi[r]
        st["out"] = torch.empty_like(st["x"])
    else:
        st["v"] = _modes(u, case["nev"], g)
        t = dims[0]
        d = torch.arange(t, device=DEV)
        fall = torch.exp(-0.4 * torch.minimum(d, t - d)).to(C128).view(1, t, 1, 1, 1, 1, 1)
        st["dist"] = _gauss((4 * case["dist"],) + dims + (4, 3), g).mul_(fall)
        st["phi"] = _gauss((4 * case["noise"],) + dims + (4, 3), g).mul_(fall)
        st["phibar"] = (st["phi"] - 0.2 * _gauss(st["phi"].shape, g).mul_(fall)).contiguous()
        if case["backward"]:
            for n in ("dist", "phi", "phibar"):
                st[n].requires_grad_()
            st["w"] = _gauss((2, dlma.NPARTS, t), g).cpu()
    return st


# ---------------------------------------------------------------- the measured pass

def run(st):
    c = st["case"]
    k = c["kind"]
    if k == "solve":
        return dlma.dlma_solve(st["handles"], st["bs"], opts=st["opts"])[0]
    if k == "operator":
        return dlma.dlma_apply_dw(st["g"], st["x"], dagger=c["dagger"])
    if k == "configuration":
        g = dlma.dlma_load_gauge(st["u"], 0.121, CSW)
        return dlma.dlma_apply_dw(g, st["x"])
    if k == "gradient":
        x = dlma.dirac_solve(st["b"], st["m0"], st["g"], st["opts"])
        return (x,) + torch.autograd.grad(x, (st["b"], st["m0"]), st["w"])
    if k == "modes":
        return dlma.dlma_lap_eigs(st["g"], c["nev"], 0, c["nt"], st["v0"], tol=c["tol"], block_size=c["block"])
    if k == "project":
        return dlma.dlma_project(st["g"], 0, st["v"], st["x"], c["mode"], out=st["out"])
    if not c["backward"]:
        return dlma.dlma_correlators(st["g"], 0, st["v"], st["dist"], st["phi"], st["phibar"], ndil=c["ndil"])
    corr = dlma.correlators(st["dist"], st["phi"], st["phibar"], st["g"], 0, st["v"], c["ndil"])
    return (corr,) + torch.autograd.grad(corr, (st["dist"], st["phi"], st["phibar"]), st["w"])


def work(case):
    """Inputs read once, outputs written once; the operations of the definition (for a solve: 58
    applications of the even-odd operator, what a Krylov method needs to 1e-10 on these fields)."""
    k = case["kind"]
    if k == "solve":
        b = f = 0
        for d, m, n, p in _parts(case):
            v, r = math.prod(d), 4 * m + 8 * n + p
            b += v * (1152 + 384 * r)
            f += 58 * v * r * (1320 + 504)
        return {"bytes": b, "flops": f}
    v = _volume(case["lat"])
    if k in ("operator", "configuration"):
        return {"bytes": v * (1152 + 384 * case["rhs"]),
                "flops": v * (1320 + 504) * case["rhs"] + (v * 24 * 3 * 198 if k == "configuration" else 0)}
    if k == "gradient":
        return {"bytes": v * (1152 + 4 * 192 * case["rhs"]), "flops": 2 * 58 * v * case["rhs"] * (1320 + 504)}
    t = _dims(case["lat"])[0]
    l3 = v // t
    if k == "modes":  # the subspace of 300 applications of the Laplacian
        return {"bytes": case["nt"] * l3 * (432 + 48 * case["nev"]), "flops": case["nt"] * l3 * 300 * 420}
    if k == "project":
        return {"bytes": l3 * 48 * case["nev"] + case["rhs"] * 192 * (v + l3), "flops": 2 * 8 * 12 * l3 * case["nev"] * case["rhs"]}
    nf = 4 * case["dist"] + 8 * case["noise"]
    b = 48 * v * case["nev"] + 192 * v * nf * (2 if case["backward"] else 1)
    f = 8 * 12 * v * case["nev"] * nf + 8 * 12 * 16 * v * nf
    return {"bytes": b, "flops": f * (2 if case["backward"] else 1)}


# ---------------------------------------------------------------- 64-bit restatement

AXIS = (1, 4, 3, 2)  # array axis of direction mu in a spinor [n, t, z, y, x, 4, 3]


def _gammas():
    s = torch.tensor([[[0, 1], [1, 0]], [[0, -1j], [1j, 0]], [[1, 0], [0, -1]]], dtype=C128)
    g = torch.zeros(5, 4, 4, dtype=C128)
    g[0, :2, 2:] = g[0, 2:, :2] = -torch.eye(2, dtype=C128)
    for k in range(3):
        g[k + 1, :2, 2:] = -1j * s[k]
        g[k + 1, 2:, :2] = 1j * s[k]
    g[4] = torch.diag(torch.tensor([1, 1, -1, -1], dtype=C128))
    return g.to(DEV)


def _clover(u, kappa):
    """A(x) as 12x12 matrices [t, z, y, x, 4, 3, 4, 3]."""
    g = _gammas()
    ax = (0, 3, 2, 1)
    link = [u[..., mu, :, :] for mu in range(4)]
    up = lambda f, mu: torch.roll(f, -1, ax[mu])  # noqa: E731
    dn = lambda f, mu: torch.roll(f, 1, ax[mu])   # noqa: E731
    a = torch.zeros(tuple(u.shape[:4]) + (4, 3, 4, 3), dtype=C128, device=DEV)
    for s in range(4):
        for c in range(3):
            a[..., s, c, s, c] = 1 / (2 * kappa)
    for mu in range(4):
        for nu in range(mu + 1, 4):
            p = _mul(_mul(link[mu], up(link[nu], mu)), _mul(link[nu], up(link[mu], nu)).mH)
            # the other three leaves, each at the corner y that its links start from, moved to x
            h = _mul(link[nu].mH, _mul(link[mu], up(link[nu], mu)))
            q = p + dn(_mul(h, up(link[mu], nu).mH), nu)
            h = _mul(_mul(up(link[nu], mu), up(link[mu], nu).mH), _mul(link[nu].mH, link[mu]))
            q = q + dn(h, mu)
            h = _mul(_mul(up(link[mu], nu).mH, link[nu].mH), _mul(link[mu], up(link[nu], mu)))
            q = q + dn(dn(h, mu), nu)
            f = (q - q.mH) / 8
            sigma = 0.5j * (g[mu] @ g[nu] - g[nu] @ g[mu])
            for s in range(4):
                for r in range(4):
                    if sigma[s, r] != 0:
                        a[..., s, :, r, :] += CSW * 0.5j * sigma[s, r] * f
    return a


def _dirac(u, a, x, dagger=False):
    g = _gammas()
    if dagger:
        x = x * torch.tensor([1, 1, -1, -1], device=DEV).view(4, 1)
    out = sum(a[..., s, c][None] * x[..., s, c, None, None] for s in range(4) for c in range(3))
    for mu in range(4):
        um = u[..., mu, :, :][..., None, :, :]  # [.., spin, a, b]
        perm = [int(torch.argmax(g[mu, s].abs())) for s in range(4)]
        ph = torch.stack([g[mu, s, perm[s]] for s in range(4)]).view(4, 1)
        f = torch.roll(x, -1, AXIS[mu])
        f = f - ph * f[..., perm, :]
        out -= 0.5 * sum(um[..., :, b] * f[..., b, None] for b in range(3))
        f = sum(um[..., b, :].conj() * x[..., b, None] for b in range(3))
        out -= 0.5 * torch.roll(f + ph * f[..., perm, :], 1, AXIS[mu])
    if dagger:
        out = out * torch.tensor([1, 1, -1, -1], device=DEV).view(4, 1)
    return out


def _invert(u, a, b, dagger=False):
    """D x = b by BiCGStab to a residual of 1e-14, restarted once."""
    dot = lambda p, q: (p.conj() * q).flatten(1).sum(1).view(-1, 1, 1, 1, 1, 1, 1)  # noqa: E731
    x = torch.zeros_like(b)
    for _ in range(2):
        r = b - _dirac(u, a, x, dagger)
        goal = 1e-14 ** 2 * dot(b, b).real
        rh = r + 0.3 * r.abs().amax() * _gauss(r.shape[1:], _gen(9))
        p, rho = r.clone(), dot(rh, r)
        for _ in range(250):
            live = dot(r, r).real > goal
            if not bool(live.any()):
                break
            v = _dirac(u, a, p, dagger)
            alpha = torch.where(live, rho / dot(rh, v), 0)
            s = r - alpha * v
            t = _dirac(u, a, s, dagger)
            omega = torch.where(live, dot(t, s) / dot(t, t), 0)
            x += alpha * p + omega * s
            r = torch.where(live, s - omega * t, r)
            new = dot(rh, r)
            beta = torch.where(live, new / rho * alpha / omega, 0)
            p = torch.where(live, r + beta * (p - omega * v), p)
            rho = new
    return x


def _low_modes(u, nev, v0):
    """The nev lowest modes of -lap by filtered subspace iteration, largest component real and positive."""
    n = 3 * math.prod(u.shape[1:4])
    kb = min(n, nev + max(12, nev // 2))
    v = _gauss((u.shape[0], kb) + tuple(u.shape[1:4]) + (3,), _gen(4))
    v = _orthonormal(v)
    for it in range(60):
        w = -_laplacian(u, v)
        h = v.flatten(2).conj() @ w.flatten(2).transpose(-1, -2).contiguous()
        lam, z = torch.linalg.eigh(0.5 * (h + h.mH))
        v = (z.transpose(-1, -2).contiguous() @ v.flatten(2)).reshape(v.shape)
        w = (z.transpose(-1, -2).contiguous() @ w.flatten(2)).reshape(v.shape)
        res = (w - lam.view(*lam.shape, 1, 1, 1, 1) * v).flatten(2).abs().square().sum(-1).sqrt()[:, :nev].max()
        if float(res) < 3e-14 or kb == n or it == 59:
            break
        cut = min(float(lam[:, -1].max()), 11.5)
        c, e = 0.5 * (cut + 12), 0.5 * (12 - cut)
        deg = 8
        while deg < 60 and math.cosh((deg + 1) * math.acosh(max((c - float(lam.min())) / e, 1.0))) < 1e7:
            deg += 1
        p, q = v, (c * v + _laplacian(u, v)) / e
        for _ in range(deg - 1):
            p, q = q, 2 * (c * q + _laplacian(u, q)) / e - p
        v = _orthonormal(q / q.flatten(2).abs().square().sum(-1).sqrt().view(*lam.shape, 1, 1, 1, 1))
    v, lam = v[:, :nev].flatten(2), lam[:, :nev]
    m = v.abs()
    first = (m >= m.amax(-1, keepdim=True) - 1e-10).to(torch.int8).argmax(-1, keepdim=True)
    top = v.gather(-1, first)
    v = v * (top.conj() / top.abs())
    return v.reshape(u.shape[0], nev, *u.shape[1:4], 3), -lam


def _pieces(case, v, dist, phi, phibar):
    """The correlator pieces [2, 7, t] from the definition, source timeslice 0."""
    g = _gammas()
    t = v.shape[0]
    nev = case["nev"]
    vm = v.reshape(t, nev, -1)

    def columns(f):  # [groups, 4, t, site, spin, colour] -> [t, (site, colour), groups, (label, spin)]
        f = f.reshape(-1, 4, t, f[0].numel() // t // 12, 4, 3)
        return f.permute(2, 3, 5, 0, 1, 4).reshape(t, vm.shape[2], -1, 16)

    def grams(a, b):  # sums over groups of <A_(s', a), B_(s, b)>, whole and projected
        full = proj = 0
        for i in range(a.shape[2]):
            p, q = a[:, :, i].contiguous(), b[:, :, i].contiguous()
            full = full + p.mH.contiguous() @ q
            vp, vq = vm.conj() @ p, vm.conj() @ q
            proj = proj + vp.mH.contiguous() @ vq
        return full.reshape(t, 4, 4, 4, 4), proj.reshape(t, 4, 4, 4, 4)

    def trace(gram, gam):
        m, n = g[4] @ gam, gam @ g[4]
        return (gram * n.T.reshape(1, 4, 1, 4, 1) * m.reshape(1, 1, 4, 1, 4)).sum((1, 2, 3, 4))

    d, f, fb = columns(dist), columns(phi), columns(phibar)
    nr = case["noise"] // case["ndil"]
    (d1, dp), (f1, fp), (b1, bp) = grams(d, d), grams(f, f), grams(fb, f)
    parts = [(b1 - bp) / nr, bp / nr, ((f1 - b1) - (fp - bp)) / nr, (fp - bp) / nr, f1 / nr, dp, d1 - dp]
    return torch.stack([torch.stack([sum(trace(p, g[i]) for i in gs) / len(gs) for p in parts]) for gs in ((4,), (1, 2, 3))])


def exact(case, seed):
    st = prepare(case, seed)
    k = case["kind"]
    if k == "solve":
        if sum(math.prod(d) * (4 * m + 8 * n + p) for d, m, n, p in _parts(case)) > 20_000_000:
            return None
        return [_invert(u, _clover(u, case["kappa"]), b) for u, b in zip(st["us"], st["bs"])]
    u = st["u"]
    if k in ("operator", "configuration"):
        a = _clover(u, 0.121)
        return torch.cat([_dirac(u, a, x[None], case.get("dagger", False)) for x in st["x"]])
    if k == "gradient":
        a = _clover(u, case["kappa"])
        x = _invert(u, a, st["b"].detach())
        gb = _invert(u, a, st["w"], dagger=True)
        return x, gb, -(gb.conj() * x).sum().real.cpu()
    if k == "modes":
        v, lam = _low_modes(u[:case["nt"]], case["nev"], st["v0"])
        return v, lam.cpu().numpy()
    if k == "project":
        f = st["v"].flatten(1)
        out = torch.zeros_like(st["x"])
        x = st["x"][:, 0].permute(0, 4, 1, 2, 3, 5).reshape(-1, f.shape[1])
        p = (x @ f.conj().T.contiguous()) @ f
        p = (x - p if case["mode"] else p).reshape(case["rhs"], 4, *st["x"].shape[2:5], 3)
        out[:, 0] = p.permute(0, 2, 3, 4, 1, 5)
        return out
    corr = _pieces(case, st["v"], st["dist"], st["phi"], st["phibar"])
    if case["backward"]:
        return (corr.detach().cpu(),) + torch.autograd.grad(corr, (st["dist"], st["phi"], st["phibar"]), st["w"].to(DEV))
    corr = corr.cpu().numpy()
    return {n: {p: corr[i, j] for j, p in enumerate(dlma.PART_NAMES)} for i, n in enumerate(dlma.GAMMA_NAMES)}
