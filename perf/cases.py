"""Performance cases of the library's public entry points.

listed() names a dozen calls over the sizes that this repository's own
workloads and tests use: single operator applications (the building block of
any solver a caller writes), the layout conversions at either end of a
program, the overlap apply in its solver forms, the shifted solutions, the
Lanczos sign function and the Wilson solve.  draw(rng) gives further calls of the same ranges.
A case is a dict of plain values; prepare(case, seed) makes its inputs on the
GPU, run(state) is one pass, work(case) the bytes and operations of the
problem and exact(case, seed) the result in 64 bits by plain torch.

Inputs follow the workload recipe: links exp(i eps0 H) of Gaussian Hermitian
H, two stout smearing steps, Gaussian or point sources, rho = 1.6.  Outputs
are the library's packed fields seen as their stored numbers, without the
padding elements (the layouts are those that ovl.h states).
"""
import math

import numpy as np
import torch

import paper_1410_7170_amd as ovl

RHO = 1.6
EPS0 = 0.3
RHO_STOUT = 0.1
# |Q| of these fields lies in about [0.40, 6.4]; the bounds that a Lanczos run
# with the usual margins gives
INTERVAL = (0.36, 6.75)
PREC = {"f64": ovl.F64, "f32": ovl.F32, "f16s": ovl.F16S}
REAL_BYTES = {"f64": 8, "f32": 4, "f16s": 2}


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # a Q^2 application on the smallest lattice in use (dense checks, unit
        # tests, inner loops over small systems): launch latency
        dict(name="q2 f64 4^4", kind="operator", op="q2", prec="f64", nrhs=1, dims="4x4x4x4"),
        # FP16 storage with per-site scales, three fields on a lattice whose
        # spatial extents fit no power of two
        dict(name="q f16s 20x14x18x10 x3", kind="operator", op="q", prec="f16s", nrhs=3, dims="20x14x18x10"),
        # the operator in double precision at the benchmark's size: residuals,
        # eigensolvers, defect corrections
        dict(name="wilson f64 32^3x64", kind="operator", op="wilson", prec="f64", nrhs=1, dims="64x32x32x32"),
        # a propagator's twelve spin-colour sources through the FP32 operator
        dict(name="wilson f32 24^3x48 x12", kind="operator", op="wilson", prec="f32", nrhs=12, dims="48x24x24x24"),
        # reading a configuration and a source in, writing a result out
        dict(name="pack 32^3x64", kind="pack", nrhs=1, dims="64x32x32x32"),
        # the overlap apply of unit tests and tiny systems, default parameters
        dict(name="overlap f64 8x4^3", kind="overlap", form="f64", nrhs=1, poles=20, tol=1e-12, dims="8x4x4x4"),
        # every shifted solution (not only their sum), blocked form, ragged extents
        dict(name="multishift 16x12x8x6", kind="multishift", nrhs=1, poles=12, tol=1e-10, dims="16x12x8x6"),
        # the overlap apply inside an outer solver on a medium lattice
        dict(name="overlap mixed 16^3x32", kind="overlap", form="mixed", nrhs=1, poles=20, tol=1e-10,
             dims="32x16x16x16"),
        # the benchmark's workload
        dict(name="overlap mixed 32^3x64", kind="overlap", form="mixed", nrhs=1, poles=20, tol=1e-10,
             dims="64x32x32x32"),
        # twelve point sources in one call
        dict(name="overlap mixed 24^3x48 x12", kind="overlap", form="mixed", nrhs=12, poles=20, tol=1e-10,
             dims="48x24x24x24"),
        # sign(Q) by the two-pass Lanczos method
        dict(name="lanczos sign 16^3x32", kind="lanczos", nrhs=1, tol=1e-10, dims="32x16x16x16"),
        # the Wilson solve of the outer solver's preconditioner, to full accuracy
        dict(name="wilson solve 32^3x64", kind="solve", m0=-0.5, nrhs=1, tol=1e-10, dims="64x32x32x32"),
    ]


def _dims(case):
    return tuple(int(v) for v in case["dims"].split("x"))


def _volume(case):
    return math.prod(_dims(case))


def draw(rng):
    kind = rng.choice(["operator"] * 4 + ["overlap"] * 3 + ["solve", "lanczos", "multishift", "pack"])

    def dims(lo, hi):
        s = lo * (hi / lo) ** rng.random()
        even = lambda v, top: int(min(top, max(2, 2 * round(v / 2))))  # noqa: E731
        d = [even(s * rng.uniform(1.0, 2.2), 64)] + [even(s * rng.uniform(0.8, 1.2), 32) for _ in range(3)]
        return "x".join(str(v) for v in d)

    def fields(case, most):
        v = _volume(case)
        return max(1, min(rng.choice([1, 1, 1, 2, 3, 4, 6, 12]), most // v))

    if kind == "operator":
        case = dict(kind=kind, op=rng.choice(["wilson", "q", "q2"]), prec=rng.choice(["f64", "f64", "f32", "f32", "f16s"]),
                    dims=dims(4, 30))
        case["nrhs"] = fields(case, 8 << 20)
    elif kind == "pack":
        case = dict(kind=kind, dims=dims(6, 30))
        case["nrhs"] = fields(case, 2 << 20)
    elif kind == "overlap":
        case = dict(kind=kind, form=rng.choice(["f64", "f64 blocked", "mixed", "mixed"]), poles=rng.choice([16, 20, 24]),
                    tol=1e-10, dims=dims(4, 22))
        case["nrhs"] = fields(case, 1 << 19)
    elif kind == "multishift":
        case = dict(kind=kind, poles=rng.choice([4, 8, 12, 20]), tol=1e-10, dims=dims(4, 14))
        case["nrhs"] = fields(case, 1 << 17)
    elif kind == "lanczos":
        case = dict(kind=kind, tol=1e-10, dims=dims(4, 18))
        case["nrhs"] = fields(case, 1 << 18)
    else:
        case = dict(kind=kind, m0=rng.choice([-0.5, -0.2, 0.0]), tol=1e-10, dims=dims(4, 26))
        case["nrhs"] = min(2, fields(case, 1 << 20))
    return case


# ------------------------------------------------------------------ inputs
def _mul(a, b):
    """Products of 3x3 matrices over leading axes."""
    return (a.unsqueeze(-1) * b.unsqueeze(-3)).sum(-2)


def _dag(a):
    return a.transpose(-1, -2).conj()


def _exp(x):
    """exp of small anti-Hermitian matrices: Taylor polynomial of x/16, squared four times."""
    x = x / 16
    one = torch.eye(3, dtype=x.dtype, device=x.device)
    out = one + x / 10
    for n in range(9, 0, -1):
        out = one + _mul(x, out) / n
    for _ in range(4):
        out = _mul(out, out)
    return out


def _su3(u):
    """Rows 0 and 1 orthonormalised, row 2 the conjugate of their cross product."""
    a = u[..., 0, :]
    a = a / a.abs().square().sum(-1, keepdim=True).sqrt()
    b = u[..., 1, :]
    b = b - (a.conj() * b).sum(-1, keepdim=True) * a
    b = b / b.abs().square().sum(-1, keepdim=True).sqrt()
    return torch.stack([a, b, _row2(a, b)], -2)


def _row2(a, b):
    return (a[..., [1, 2, 0]] * b[..., [2, 0, 1]] - a[..., [2, 0, 1]] * b[..., [1, 2, 0]]).conj()


def _links(dims, seed):
    """The smeared gauge field, (L0, L1, L2, L3, 4, 3, 3) complex128 on the GPU."""
    g = torch.Generator(device="cuda").manual_seed(2 * seed + 1)
    a = torch.randn(*dims, 4, 3, 3, dtype=torch.complex128, device="cuda", generator=g)
    h = (a + _dag(a)) / 2
    h = h - torch.diag_embed(h.diagonal(dim1=-2, dim2=-1).sum(-1, keepdim=True).expand(*dims, 4, 3) / 3)
    u = _su3(_exp(1j * EPS0 * h))
    del a, h
    for _ in range(2):
        new = []
        for mu in range(4):
            um = u[..., mu, :, :]
            staples = torch.zeros_like(um)
            for nu in range(4):
                if nu == mu:
                    continue
                un = u[..., nu, :, :]
                un_mu = un.roll(-1, mu)   # U_nu(x + mu)
                staples += _mul(_mul(un, um.roll(-1, nu)), _dag(un_mu))
                staples += _mul(_mul(_dag(un), um), un_mu).roll(1, nu)
            m = _mul(staples, _dag(um))
            z = (m - _dag(m)) / 2
            z = z - torch.diag_embed(z.diagonal(dim1=-2, dim2=-1).sum(-1, keepdim=True).expand(*dims, 3) / 3)
            new.append(_su3(_mul(_exp(RHO_STOUT * z), um)))
        u = torch.stack(new, -3)
    return u.contiguous()


def _sources(case, seed):
    """(nrhs, V, 4, 3) complex128: Gaussian, or the twelve point sources of a site."""
    V, n = _volume(case), case["nrhs"]
    g = torch.Generator(device="cuda").manual_seed(2 * seed)
    if case["kind"] == "overlap" and n == 12:
        site = int(torch.randint(V, (1,), device="cuda", generator=g))
        b = torch.zeros(12, V, 12, dtype=torch.complex128, device="cuda")
        b[torch.arange(12), site, torch.arange(12)] = 1
        return b.view(12, V, 4, 3)
    return torch.randn(n, V, 4, 3, dtype=torch.complex128, device="cuda", generator=g)


# ------------------------------------------------------------------ packed fields
def _numbers(lat, s):
    """A packed field set's stored numbers, without the padding elements."""
    n, Vh = s.nrhs, lat.V // 2
    if s.prec == ovl.F64:
        return [s.data.view(torch.float64).view(n, 2, 12, -1, 2)[..., :Vh, :]]
    if s.prec == ovl.F32:
        return [s.data.view(torch.float32).view(n, 2, 6, -1, 4)[..., :Vh, :]]
    return [s.data.view(torch.float16).view(n, 2, 3, -1, 8)[..., :Vh, :], s.scale.view(n, 2, -1)[..., :Vh]]


def _link_numbers(lat, U):
    Vh = lat.V // 2
    kinds = {ovl.F64: (torch.float64, 6, 2), ovl.F32: (torch.float32, 3, 4), ovl.F16S: (torch.float16, 3, 4)}
    return [U.bufs[p].view(t).view(2, 4, k, -1, w)[..., :Vh, :] for p, (t, k, w) in kinds.items()]


def _halves(dims):
    """The lexicographic sites of parity 0 and of parity 1, in packed order."""
    x = [torch.arange(n, device="cuda").view([-1 if m == k else 1 for k in range(4)]) for m, n in enumerate(dims)]
    odd = ((x[0] + x[1] + x[2] + x[3]) % 2).reshape(-1)
    lex = torch.arange(odd.numel(), device="cuda")
    return lex[odd == 0], lex[odd == 1]


def _as_packed(dims, f, prec):
    """What _numbers gives for the field f (nrhs, V, 4, 3), in 64 bits."""
    n = f.shape[0]
    per = {"f64": 2, "f32": 4, "f16s": 8}[prec]
    out, scales = [], []
    for sites in _halves(dims):
        v = torch.view_as_real(f.reshape(n, -1, 12)[:, sites].contiguous()).reshape(n, len(sites), 24)
        if prec == "f16s":
            top = v.abs().amax(-1)
            scales.append(torch.where(top > 0, top, torch.ones_like(top)))
            v = v / scales[-1].unsqueeze(-1)
        out.append(v.view(n, len(sites), 24 // per, per).transpose(1, 2))
    return [torch.stack(out, 1)] + ([torch.stack(scales, 1)] if prec == "f16s" else [])


# ------------------------------------------------------------------ a pass
def _params(case):
    form = {"f64": {}, "f64 blocked": dict(block=16), "mixed": dict(mode=ovl.SOLVE_MIXED)}
    kind = case["kind"]
    if kind == "overlap":
        return ovl.default_params(tol=case["tol"], **form[case["form"]])
    if kind == "multishift":
        return ovl.default_params(tol=case["tol"], block=8)
    if kind == "lanczos":
        return ovl.default_params(tol=case["tol"], mode=ovl.SOLVE_LANCZOS)
    return ovl.default_params(tol=case["tol"], even_odd=1)


def prepare(case, seed):
    dims, kind = _dims(case), case["kind"]
    lat = ovl.Lattice(dims)
    links = _links(dims, seed).view(lat.V, 4, 3, 3)
    src = _sources(case, seed)
    if kind == "pack":
        return dict(case=case, lat=lat, links=links, src=src)
    prec = PREC[case.get("prec", "f64")]
    precs = (prec,) if kind == "operator" else (ovl.F64, ovl.F32)
    s = dict(case=case, lat=lat, U=ovl.Gauge(lat, links, precs), b=ovl.Spinor.from_canonical(lat, src, prec))
    count = case["nrhs"] * (case["poles"] if kind == "multishift" else 1)
    s["x"] = ovl.Spinor(lat, prec, count)
    s["out"] = _numbers(lat, s["x"])
    if kind == "operator":
        s["ws"] = ovl.workspace(lat, ovl.OP_Q2, prec, case["nrhs"]) if case["op"] == "q2" else None
        return s
    s["prm"] = _params(case)
    if kind != "solve":
        s["shifts"], s["weights"], _ = ovl.zolotarev(*INTERVAL, case.get("poles", 20))
    # the workspace is kept between calls where three of them fit beside each
    # other, else the call takes it from torch's allocator
    if kind == "solve":
        s["ws"] = ovl.workspace(lat, ovl.OP_WILSON_SOLVE, ovl.F64, case["nrhs"], 0, s["prm"])
    else:
        need = ovl.workspace_bytes(lat, ovl.OP_MSCG, ovl.F64, case["nrhs"], len(s["shifts"]), s["prm"])
        s["ws"] = torch.empty(need, dtype=torch.uint8, device="cuda") if need < 50 << 30 else None
    return s


def run(s):
    case = s["case"]
    kind, lat = case["kind"], s["lat"]
    if kind == "pack":
        U = ovl.Gauge(lat, s["links"])
        b = ovl.Spinor.from_canonical(lat, s["src"], ovl.F64)
        c = ovl.Spinor.from_canonical(lat, s["src"], ovl.F32)
        return _link_numbers(lat, U) + _numbers(lat, b) + _numbers(lat, c) + [b.to_canonical()]
    U, b, x, ws = s["U"], s["b"], s["x"], s["ws"]
    if kind == "operator":
        if case["op"] == "q2":
            ovl.q2_apply(lat, U, -RHO, 0.25, b, x, ws)
        elif case["op"] == "q":
            ovl.q_apply(lat, U, -RHO, b, x)
        else:
            ovl.wilson_apply(lat, U, -RHO, b, x)
    elif kind == "overlap":
        ovl.overlap_apply(lat, U, RHO, s["shifts"], s["weights"], b, x, s["prm"], ws)
    elif kind == "lanczos":
        ovl.sign_q_apply(lat, U, -RHO, s["shifts"], s["weights"], b, x, s["prm"], ws)
    elif kind == "multishift":
        ovl.multishift_cg(lat, U, -RHO, s["shifts"], None, b, x, s["prm"], ws)
    else:
        ovl.wilson_solve(lat, U, case["m0"], b, x, s["prm"], ws)
    return s["out"]


# ------------------------------------------------------------------ the problem's size
# operator applications that a Krylov method spends to 1e-10 on these fields
# (the Q^2 steps of the multishift CG, the steps of the Lanczos method, the
# steps of the reduced Wilson solve)
STEPS = {"overlap": 160, "multishift": 150, "lanczos": 320, "solve": 48}


def work(case):
    V, n, kind = _volume(case), case["nrhs"], case["kind"]
    real = REAL_BYTES[case.get("prec", "f64")]
    spinor, link = 24 * real + (4 if real == 2 else 0), 4 * 12 * real   # bytes a site
    hop = 1320 + 48   # operations a site of one D_W
    if kind == "operator":
        return {"bytes": V * (2 * n * spinor + link), "flops": V * n * hop * (2 if case["op"] == "q2" else 1)}
    if kind == "pack":
        return {"bytes": V * (4 * 18 * 8 + 4 * 12 * (8 + 4 + 2) + n * (192 + 192 + 96 + 192)), "flops": 0}
    bytes_ = V * (link + n * (spinor + spinor * (case["poles"] if kind == "multishift" else 1)))
    return {"bytes": bytes_, "flops": V * n * STEPS[kind] * 2 * hop}


# ------------------------------------------------------------------ 64 bits, plain torch
# gamma_mu in the chiral basis, one entry a row: (column, phase)
GAMMA = [([2, 3, 0, 1], [1, 1, 1, 1]), ([3, 2, 1, 0], [-1j, -1j, 1j, 1j]), ([3, 2, 1, 0], [-1, 1, 1, -1]),
         ([2, 3, 0, 1], [-1j, 1j, 1j, -1j])]


def _wilson(u, f, m0):
    """D_W(m0) f for f (nrhs, L0, L1, L2, L3, 4, 3): antiperiodic in axis 0."""
    out = (m0 + 4) * f

    def times(m, v):   # 3x3 matrices on the colours of every spin
        return (m.unsqueeze(-3) * v.unsqueeze(-2)).sum(-1)

    for mu in range(4):
        col, phase = GAMMA[mu]
        phase = torch.tensor(phase, dtype=f.dtype, device=f.device).view(4, 1)
        um = u[..., mu, :, :]
        up = f.roll(-1, mu + 1)
        if mu == 0:
            up[:, -1] = -up[:, -1]
        up = up - phase * up[..., col, :]
        down = f + phase * f[..., col, :]
        for r in range(f.shape[0]):
            out[r] -= times(um, up[r]) / 2
            d = times(_dag(um), down[r]).roll(1, mu)
            if mu == 0:
                d[0] = -d[0]
            out[r] -= d / 2
    return out


def _q(u, f, m0):
    out = _wilson(u, f, m0)
    out[..., :2, :] *= -1
    return out


def _zolotarev(lo, hi, n):
    """Poles and weights of x sum w/(x^2 + s) ~ sign(x) on [lo, hi]: Zolotarev's
    elliptic formula, sn by the arithmetic-geometric mean."""
    k1 = lo / hi                                  # complementary modulus
    a, b, c = [1.0], [k1], [math.sqrt(1 - k1 * k1)]
    while c[-1] > 1e-17:
        a0, b0 = a[-1], b[-1]
        a.append((a0 + b0) / 2)
        b.append(math.sqrt(a0 * b0))
        c.append((a0 - b0) / 2)
    K = math.pi / (2 * a[-1])
    coef = []
    for j in range(1, 2 * n):
        phi = 2 ** (len(a) - 1) * a[-1] * j * K / (2 * n)
        for i in range(len(a) - 1, 0, -1):
            phi = (phi + math.asin(c[i] / a[i] * math.sin(phi))) / 2
        coef.append(math.tan(phi) ** 2 * lo * lo)
    poles, zeros = np.array(coef[0::2]), np.array(coef[1::2])
    w = np.array([np.prod((zeros - p) / np.delete(poles - p, i)) for i, p in enumerate(poles)])
    x = np.exp(np.linspace(math.log(lo), math.log(hi), 40001))
    r = x * sum(wi / (x * x + p) for wi, p in zip(w, poles))
    return poles, w * 2 / (r.max() + r.min())


def _shifted(u, b, m0, shifts, tol=2e-14, most=600):
    """All solutions of (Q^2 + s) x = b by multishift CG (one field)."""
    base = min(shifts)
    x = [torch.zeros_like(b) for _ in shifts]
    p = [b.clone() for _ in shifts]
    r = b.clone()
    rr = bb = float(torch.vdot(b.flatten(), b.flatten()).real)
    j0 = int(np.argmin(shifts))
    z, z_old = np.ones(len(shifts)), np.ones(len(shifts))
    alpha_old, beta = 1.0, 0.0
    for _ in range(most):
        t = _q(u, p[j0], m0)
        alpha = rr / (float(torch.vdot(t.flatten(), t.flatten()).real)
                      + base * float(torch.vdot(p[j0].flatten(), p[j0].flatten()).real))
        d = np.array(shifts) - base
        z_new = z * z_old * alpha_old / (alpha * beta * (z_old - z) + z_old * alpha_old * (1 + alpha * d))
        r.add_(_q(u, t, m0).add_(p[j0], alpha=base), alpha=-alpha)
        new = float(torch.vdot(r.flatten(), r.flatten()).real)
        beta = new / rr
        for j in range(len(shifts)):
            if abs(z[j]) * math.sqrt(rr) < 1e-16 * math.sqrt(bb):
                continue
            x[j].add_(p[j], alpha=alpha * z_new[j] / z[j])
            p[j].mul_(beta * (z_new[j] / z[j]) ** 2).add_(r, alpha=z_new[j])
        z_old = np.where(np.abs(z_new) > 1e-200, z, z_old)
        z = np.where(np.abs(z_new) > 1e-200, z_new, z)
        alpha_old, rr = alpha, new
        if rr <= tol * tol * bb:
            break
    return x


def _solve(u, b, m0, tol=2e-14, most=600):
    """D_W(m0) x = b by CG on the normal equations."""
    g5 = torch.tensor([-1, -1, 1, 1], dtype=b.dtype, device=b.device).view(4, 1)
    x, r = torch.zeros_like(b), b.clone()
    s = g5 * _wilson(u, g5 * r, m0)
    p, gamma = s.clone(), float(s.abs().square().sum())
    stop = tol * tol * float(b.abs().square().sum())
    for _ in range(most):
        q = _wilson(u, p, m0)
        alpha = gamma / float(q.abs().square().sum())
        x.add_(p, alpha=alpha)
        r.add_(q, alpha=-alpha)
        if float(r.abs().square().sum()) <= stop:
            break
        s = g5 * _wilson(u, g5 * r, m0)
        new = float(s.abs().square().sum())
        p = s + (new / gamma) * p
        gamma = new
    return x


def exact(case, seed):
    dims, kind, n = _dims(case), case["kind"], case["nrhs"]
    V = _volume(case)
    if kind in ("overlap", "lanczos", "multishift", "solve") and V * n > 2200000:
        return None   # minutes of plain torch
    u, b = _links(dims, seed), _sources(case, seed)
    if kind == "pack":
        rows = torch.view_as_real(u.view(V, 4, 3, 3)[:, :, :2].contiguous()).reshape(V, 4, 12)
        links = []
        for per in (2, 4, 4):
            halves = [rows[s].view(len(s), 4, 12 // per, per).permute(1, 2, 0, 3) for s in _halves(dims)]
            links.append(torch.stack(halves, 0))
        return links + _as_packed(dims, b, "f64") + _as_packed(dims, b, "f32") + [b]
    f = b.view(n, *dims, 4, 3)
    if kind == "operator":
        prec = case["prec"]
        if prec != "f64":   # the stored inputs
            t = torch.float32 if prec == "f32" else torch.float16
            v = torch.view_as_real(f)
            if prec == "f16s":
                top = v.abs().flatten(-3).amax(-1).float().double().view(n, *dims, 1, 1, 1)
                v = (v / top).to(t).double() * top
            else:
                v = v.to(t).double()
            f = torch.view_as_complex(v.contiguous())
            u2 = torch.view_as_complex(torch.view_as_real(u[..., :2, :].contiguous()).to(t).double())
            u = torch.cat([u2, _row2(u2[..., 0, :], u2[..., 1, :]).unsqueeze(-2)], -2)
        if case["op"] == "wilson":
            out = _wilson(u, f, -RHO)
        elif case["op"] == "q":
            out = _q(u, f, -RHO)
        else:
            out = _q(u, _q(u, f, -RHO), -RHO) + 0.25 * f
        return _as_packed(dims, out.reshape(n, V, 4, 3), prec)
    if kind == "solve":
        out = [_solve(u, f[r:r + 1], case["m0"]) for r in range(n)]
        return _as_packed(dims, torch.cat(out).reshape(n, V, 4, 3), "f64")
    shifts, weights = _zolotarev(*INTERVAL, case.get("poles", 20))
    out = []
    for r in range(n):
        xs = _shifted(u, f[r:r + 1], -RHO, list(shifts))
        if kind == "multishift":
            out.append(torch.stack(xs))   # (poles, 1, ...)
            continue
        y = torch.zeros_like(xs[0])
        for x, w in zip(xs, weights):
            y.add_(x, alpha=w)
        out.append(RHO * (f[r:r + 1] + _wilson(u, y, -RHO)) if kind == "overlap" else _q(u, y, -RHO))
    if kind == "multishift":   # field index shift * nrhs + source
        full = torch.cat(out, 1).reshape(case["poles"] * n, V, 4, 3)
    else:
        full = torch.cat(out).reshape(n, V, 4, 3)
    return _as_packed(dims, full, "f64")
