"""The workloads whose speed this framework is measured by.

Each case is one pass of what a lattice program asks of the library through
`binding.Context`: applications of the staggered and Wilson operators, CG
solves (single, batched, served), the molecular-dynamics forces and a short
trajectory.  A case is a dict of plain values:

  op     dslash | cg | batch | wilson | wilson_hop | forces | md | serve
  lx ly lz lt   lattice extents (all even)
  prec   0 FP64, 1 FP32, 2 FP16 (inner precision of a mixed solve)
  links  "su3" (proj_SU3(exp(i eps H)), stored as two rows) or "fat" (the
         same links times a real factor per link, as smeared links are not
         unitary: stored as three rows)

and, by op, mass, kappa, tol, parity, nrhs and eps, the links' roughness.
Every input is drawn on the GPU from the seed.  `exact` is plain torch in
complex128.
"""

from __future__ import annotations

import math

import torch

from paper_1311_2719_amd import binding

_ROWS = {"su3": 2, "fat": 3}


def listed():
    return [
        # a small operator application on one parity, as a coarse or test lattice makes it: launch latency
        _case("dslash_f32_8", "dslash", (8, 8, 8, 8), prec=1, parity=1),
        # the operator on the largest lattice: beyond every cache
        _case("dslash_f64_32", "dslash", (32, 32, 32, 32), parity=2, eps=0.5),
        # a small solve of uneven extents on one parity with the other half reconstructed (the force solve's form)
        _case("cg_f32_6x10x14x8", "cg", (6, 10, 14, 8), prec=1, mass=0.05, parity=1, y=True, tol=1e-11),
        # the ordinary FP64 solve
        _case("cg_f64_16", "cg", (16, 16, 16, 16), mass=0.05),
        # the largest solve, in FP64 and with FP16 inner iterations
        _case("cg_f64_32", "cg", (32, 32, 32, 32), mass=0.01, eps=0.5),
        _case("cg_f16_32", "cg", (32, 32, 32, 32), prec=2, mass=0.01, eps=0.5, tol=1e-11),
        # a propagator's twelve sources in one batched solve, masses spread over a decade
        _case("batch_f32_24_x12", "batch", (24, 24, 24, 24), prec=1, mass=0.01, eps=0.5, nrhs=12, tol=1e-11),
        # requests of two resident lattices queued at once and waited for: continuous batching
        _case("serve_f32_16_8_x16", "serve", (16, 16, 16, 16), prec=1, mass=0.02, eps=0.5, nrhs=16, tol=1e-11),
        # Wilson fermions: a solve, and the operator alone on the largest lattice
        _case("wilson_16", "wilson", (16, 16, 16, 16), kappa=0.12),
        _case("wilson_hop_32", "wilson_hop", (32, 32, 32, 32), parity=2, eps=0.5),
        # one momentum kick: the gauge force, and the fermion force added to it
        _case("forces_16", "forces", (16, 16, 16, 16)),
        # a short leapfrog trajectory: forces, solves on changing links, link updates
        _case("md_f64_12x12x12x16", "md", (12, 12, 12, 16), mass=0.05, steps=3),
    ]


def _case(name, op, dims, prec=0, links="su3", eps=0.3, **kw):
    c = {"name": name} if name else {}
    c.update(op=op, lx=dims[0], ly=dims[1], lz=dims[2], lt=dims[3], prec=prec, links=links, eps=eps)
    if op in ("cg", "batch", "serve", "md"):
        c.update(mass=0.05, tol=1e-10)
    if op in ("dslash", "cg", "wilson_hop"):
        c.update(parity=2)
    c.update(kw)
    return c


def _draw_dims(rng, lo, hi):
    """Four even extents, 4 to 32, whose volume is near a log-uniform draw of [lo, hi] and not above hi."""
    while True:
        want = math.exp(rng.uniform(math.log(lo), math.log(hi)))
        side = want ** 0.25
        d = [2 * max(2, min(16, round(side * math.exp(rng.uniform(-0.45, 0.45)) / 2))) for _ in range(3)]
        last = 2 * max(2, min(16, round(want / (d[0] * d[1] * d[2]) / 2)))
        d.insert(rng.randrange(4), last)
        if lo / 2 <= d[0] * d[1] * d[2] * d[3] <= hi:
            return tuple(d)


def draw(rng):
    op = rng.choice(["dslash", "cg", "cg", "cg", "batch", "wilson", "wilson_hop", "forces", "md", "serve"])
    links = "fat" if op in ("dslash", "cg", "batch") and rng.random() < 0.25 else "su3"
    eps = round(rng.uniform(0.25, 0.5), 3)
    mass = round(math.exp(rng.uniform(math.log(0.02), math.log(0.2))), 4)
    big, mid = 32 ** 4 * 3 // 4, 24 ** 4 * 3 // 4
    if op == "dslash":
        return _case("", op, _draw_dims(rng, 256, big), prec=rng.choice([0, 0, 1]), links=links, eps=eps, parity=rng.choice([0, 1, 2, 2]))
    if op == "cg":
        parity = rng.choice([0, 1, 2, 2])
        return _case("", op, _draw_dims(rng, 512, big), prec=rng.choice([0, 1, 2]), links=links, eps=eps, mass=mass, tol=1e-11, parity=parity, y=rng.random() < 0.3)
    if op == "batch":
        return _case("", op, _draw_dims(rng, 512, mid), prec=rng.choice([0, 1, 1, 2]), links=links, eps=eps, mass=mass, nrhs=rng.randint(2, 12), tol=1e-11)
    if op == "wilson":
        return _case("", op, _draw_dims(rng, 256, 20 ** 4), eps=eps, kappa=round(rng.uniform(0.1, 0.125), 4))
    if op == "wilson_hop":
        return _case("", op, _draw_dims(rng, 256, big), eps=eps, parity=rng.choice([0, 1, 2]))
    if op == "forces":
        return _case("", op, _draw_dims(rng, 256, mid), eps=eps)
    if op == "md":
        return _case("", op, _draw_dims(rng, 256, 16 ** 4), prec=rng.choice([0, 1]), eps=eps, mass=round(rng.uniform(0.05, 0.2), 4), steps=rng.randint(1, 3), tol=1e-11)
    return _case("", op, _draw_dims(rng, 8 ** 4, 20 ** 4), prec=1, eps=eps, mass=mass, nrhs=rng.randint(4, 24), tol=1e-11)


# ---- inputs -----------------------------------------------------------------------------


def _dims(case):
    return (case["lx"], case["ly"], case["lz"], case["lt"])


def _volume(d):
    return d[0] * d[1] * d[2] * d[3]


def _mm(a, b):
    """Products of 3x3 matrices, elementwise."""
    return a[..., :, 0:1] * b[..., 0:1, :] + a[..., :, 1:2] * b[..., 1:2, :] + a[..., :, 2:3] * b[..., 2:3, :]


def _dag(a):
    return a.mH.contiguous()


def _trace(a):
    return a[..., 0, 0] + a[..., 1, 1] + a[..., 2, 2]


def _eye(device):
    return torch.eye(3, dtype=torch.complex128, device=device)


def _exp(a):
    """exp of 3x3 matrices: Taylor series of a / 16, squared four times."""
    a = a / 16
    s = _eye(a.device) + a / 12
    for k in range(11, 0, -1):
        s = _eye(a.device) + _mm(a, s) / k
    for _ in range(4):
        s = _mm(s, s)
    return s


def _su3(m):
    """Gram-Schmidt on rows 0 and 1, row 2 = conj(row 0 x row 1)."""
    r0 = m[..., 0, :] / torch.linalg.vector_norm(m[..., 0, :], dim=-1, keepdim=True)
    r1 = m[..., 1, :] - (r0.conj() * m[..., 1, :]).sum(-1, keepdim=True) * r0
    r1 = r1 / torch.linalg.vector_norm(r1, dim=-1, keepdim=True)
    return torch.stack([r0, r1, torch.linalg.cross(r0, r1).conj()], dim=-2)


def _ta(z):
    """Traceless anti-Hermitian part."""
    a = 0.5 * (z - _dag(z))
    return a - (_trace(a) / 3)[..., None, None] * _eye(z.device)


def _gauss(gen, shape):
    return torch.randn(shape, dtype=torch.complex128, device="cuda", generator=gen) * math.sqrt(2.0)  # Re, Im ~ N(0, 1)


def _links(case, d, gen):
    v = _volume(d)
    a = _gauss(gen, (v, 4, 3, 3)) / math.sqrt(2.0)
    h = 0.5 * (a + _dag(a))
    h = h - (_trace(h) / 3)[..., None, None] * _eye(h.device)
    u = _su3(_exp(1j * case["eps"] * h))
    if case["links"] == "fat":
        u = u * (1.0 + 0.1 * torch.rand((v, 4, 1, 1), dtype=torch.float64, device="cuda", generator=gen) - 0.05)
    return u.contiguous()


def _inputs(case, seed):
    """All inputs of a case, lexicographic, on the GPU."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1000003 * int(seed) + 17)
    d, op = _dims(case), case["op"]
    v = _volume(d)
    inp = {"u": _links(case, d, gen)}
    if op in ("wilson", "wilson_hop"):
        inp["b"] = _gauss(gen, (v, 4, 3))
    elif op == "batch":
        inp["bs"] = [_gauss(gen, (v, 3)) for _ in range(case["nrhs"])]
    elif op == "serve":
        d2 = _small(d)
        inp["u2"] = _links(case, d2, gen)
        inp["bs"] = [_gauss(gen, (_volume(d if i % 2 == 0 else d2), 3)) for i in range(case["nrhs"])]
    else:
        inp["b"] = _gauss(gen, (v, 3))
    if op == "md":
        inp["q"] = _ta(_gauss(gen, (v, 4, 3, 3))) / math.sqrt(2.0)  # <-tr Q^2> = 4 a link, as the heatbath gives
    return inp


def _small(d):
    """The second field of a serving case: half of each extent, even and at least 4."""
    return tuple(max(4, n // 4 * 2) for n in d)


def _masses(case):
    """Masses over a decade from the case's smallest one."""
    n, lo = case["nrhs"], case["mass"]
    return [lo * 10.0 ** (i / max(1, n - 1)) for i in range(n)]


# ---- the framework's calls ------------------------------------------------------------------


def prepare(case, seed):
    inp, d, op = _inputs(case, seed), _dims(case), case["op"]
    v = _volume(d)
    ctx = binding.Context(arena_bytes=(256 << 20) + v * (9000 if op in ("batch", "serve") else 4000))
    s = {"case": case, "ctx": ctx, "d": d}
    if op in ("wilson", "wilson_hop"):
        s["f"] = ctx.set_gauge_wilson(d, inp["u"])
        s["b"] = ctx.pack_spinor(s["f"], inp["b"])
        s["x"] = ctx.new_spinor(s["f"])
        return s
    s["f"] = ctx.set_gauge(d, inp["u"])
    if op == "dslash":
        s["b"] = ctx.pack(s["f"], inp["b"])
        if case["prec"]:
            s["b"] = ctx.convert(s["f"], s["b"], ctx.new_fermion(s["f"], case["prec"]), binding.F64, case["prec"])
        s["x"] = ctx.new_fermion(s["f"], case["prec"])
    elif op == "cg":
        s["b"], s["x"] = ctx.pack(s["f"], inp["b"]), ctx.new_fermion(s["f"])
        s["y"] = ctx.new_fermion(s["f"]) if case.get("y") else None
    elif op == "batch":
        s["bs"] = [ctx.pack(s["f"], b) for b in inp["bs"]]
        s["xs"] = [ctx.new_fermion(s["f"]) for _ in inp["bs"]]
        s["params"] = [binding.params(m, tol=case["tol"], precision=case["prec"]) for m in _masses(case)]
    elif op == "serve":
        f2 = ctx.set_gauge(_small(d), inp["u2"])
        s["fs"] = [s["f"] if i % 2 == 0 else f2 for i in range(case["nrhs"])]
        s["bs"] = [ctx.pack(f, b) for f, b in zip(s["fs"], inp["bs"])]
        s["xs"] = [ctx.new_fermion(f) for f in s["fs"]]
    elif op == "forces":
        s["u"], s["w"] = inp["u"], ctx.pack(s["f"], inp["b"])
        s["q"] = torch.zeros_like(inp["u"])
    elif op == "md":
        s["u0"], s["q0"] = inp["u"], inp["q"]
        s["u"], s["q"] = torch.empty_like(inp["u"]), torch.empty_like(inp["q"])
        s["phi"] = ctx.pseudofermion(s["f"], ctx.pack(s["f"], inp["b"]), case["mass"])
    return s


def run(s):
    c, ctx, op = s["case"], s["ctx"], s["case"]["op"]
    if op == "dslash":
        return ctx.dslash(s["f"], s["b"], s["x"], out_parity=c["parity"], precision=c["prec"])
    if op == "cg":
        ctx.cg_solve(s["f"], s["b"], s["x"], y=s["y"], mass=c["mass"], tol=c["tol"], precision=c["prec"], parity=c["parity"])
        return [s["x"]] if s["y"] is None else [s["x"], s["y"]]
    if op == "batch":
        ctx.cg_solve_batch(s["f"], s["bs"], s["xs"], s["params"])
        return s["xs"]
    if op == "serve":
        tickets = [ctx.submit(f, b, x, mass=m, tol=c["tol"], precision=c["prec"]) for f, b, x, m in zip(s["fs"], s["bs"], s["xs"], _masses(c))]
        for t in tickets:
            if ctx.wait(t)["rc"]:
                raise RuntimeError("a request failed")
            ctx.release(t)
        return s["xs"]
    if op == "wilson":
        ctx.wilson_solve(s["f"], s["b"], s["x"], c["kappa"])
        return s["x"]
    if op == "wilson_hop":
        return ctx.wilson_dslash(s["f"], s["b"], s["x"], out_parity=c["parity"])
    if op == "forces":
        ctx.gauge_force(s["d"], s["u"], 5.6, force=s["q"])
        return ctx.fermion_force(s["f"], s["w"], force=s["q"], accumulate=True)
    # md: the links before a trajectory are kept, as the accept / reject step that follows one needs them
    s["u"].copy_(s["u0"])
    s["q"].copy_(s["q0"])
    ctx.md_trajectory(s["d"], s["u"], s["q"], s["phi"], 5.6, c["mass"], 0.02, c["steps"], tol=c["tol"], precision=c["prec"])
    return [s["u"], s["q"]]


# ---- what a pass cannot do without --------------------------------------------------------------


def _iterations(case, d, mass):
    """About the CG iterations to the tolerance: from the smallest lattice momentum and the links' roughness."""
    low = mass ** 2 + math.sin(math.pi / max(4, max(d))) ** 2 * (0.35 if case["eps"] > 0.4 else 0.8)
    return max(10, 0.5 * math.log(2 / case["tol"]) * math.sqrt(4 / low))


def work(case):
    """Links count once per operator application (4 a site, two or three rows as they are stored), vectors once
    where they are read or written; a solve's iteration applies the operator twice and updates x, r and p."""
    d, op = _dims(case), case["op"]
    v, link = _volume(d), 4 * 3 * _ROWS[case["links"]]
    size = {0: 16, 1: 8, 2: 4}[case["prec"]]
    share = 1.0 if case.get("parity", 2) == 2 else 0.5
    hop = 570.0 * v  # flops of one application to every site
    if op == "dslash":
        return {"bytes": v * (link * size + 6 * size * share), "flops": hop * share}
    if op == "wilson_hop":
        return {"bytes": v * (link * 16 + 24 * 16 * share), "flops": 1320.0 * v * share}
    if op == "forces":
        return {"bytes": v * (link * 16 + 48 + 36 * 16), "flops": v * (4 * 6 * 2 * 198.0 + 4 * 200.0)}

    def solve(dd, masses, parity_share):
        n = _volume(dd)
        it = [_iterations(case, dd, m) for m in masses]
        vec = sum(it) * n * parity_share * 3 * (5 * size + 2 * (16 if size == 16 else 8))
        return {"bytes": max(it) * 2 * n * link * size + vec, "flops": sum(it) * 2 * 570.0 * n * parity_share}

    if op == "cg":
        return solve(d, [case["mass"]], share)
    if op == "batch":
        return solve(d, _masses(case), 1.0)
    if op == "serve":
        a, b = solve(d, _masses(case)[0::2], 1.0), solve(_small(d), _masses(case)[1::2], 1.0)
        return {k: a[k] + b[k] for k in a}
    if op == "wilson":
        return {"bytes": 56 * v * (4 * link * 16 + 0.5 * 12 * 16 * 10), "flops": 56 * 4 * 1320.0 * v / 2}
    one = solve(d, [case["mass"]], 0.5)
    n = case["steps"] + 1
    return {"bytes": n * (one["bytes"] + v * 36 * 16 * 6), "flops": n * (one["flops"] + v * 12000.0)}


# ---- the same results in plain torch, 64 bits ----------------------------------------------------


class _Lattice:
    """Lexicographic neighbours and the staggered factors of a lattice, antiperiodic in t."""

    def __init__(self, d):
        self.d, self.v = d, _volume(d)
        s = torch.arange(self.v, device="cuda")
        x = [s % d[0], s // d[0] % d[1], s // (d[0] * d[1]) % d[2], s // (d[0] * d[1] * d[2])]
        stride = [1, d[0], d[0] * d[1], d[0] * d[1] * d[2]]
        self.fwd = [s + torch.where(x[m] == d[m] - 1, 1 - d[m], 1) * stride[m] for m in range(4)]
        self.bwd = [s + torch.where(x[m] == 0, d[m] - 1, -1) * stride[m] for m in range(4)]
        self.odd = (x[0] + x[1] + x[2] + x[3]) % 2 == 1
        self.wrap = torch.where(x[3] == d[3] - 1, -1.0, 1.0).double()
        self.eta, phase = [], torch.zeros_like(s)
        for m in range(4):
            self.eta.append((1.0 - 2.0 * (phase % 2)).double())
            phase = phase + x[m]
        self.order = torch.cat([s[~self.odd], s[self.odd]])  # even-odd order

    def to_eo(self, lex):
        """(V, n...) -> (2, n, V/2)."""
        f = lex.reshape(self.v, -1)[self.order]
        return f.reshape(2, self.v // 2, -1).transpose(1, 2).contiguous()


def _mv(u, x):
    """u x for 3x3 matrices; x: (V, 3) or (V, 2 or 4 spins, 3)."""
    for _ in range(x.dim() - 2):
        u = u.unsqueeze(-3)
    return u[..., :, 0] * x[..., 0:1] + u[..., :, 1] * x[..., 1:2] + u[..., :, 2] * x[..., 2:3]


def _hops(lat, u, staggered):
    """Forward links with their factors, and the daggered links of the backward neighbours."""
    f, b = [], []
    for m in range(4):
        c = (0.5 * lat.eta[m] if staggered else torch.ones_like(lat.eta[m])) * (lat.wrap if m == 3 else 1.0)
        w = u[:, m] * c[:, None, None]
        f.append(w.contiguous())
        b.append(_dag(w[lat.bwd[m]]))
    return f, b


def _stag(lat, hops, x):
    f, b = hops
    out = torch.zeros_like(x)
    for m in range(4):
        out += _mv(f[m], x[lat.fwd[m]]) - _mv(b[m], x[lat.bwd[m]])
    return out


def _gammas():
    i = 1j
    g = [[[0, 0, 0, i], [0, 0, i, 0], [0, -i, 0, 0], [-i, 0, 0, 0]], [[0, 0, 0, -1], [0, 0, 1, 0], [0, 1, 0, 0], [-1, 0, 0, 0]],
         [[0, 0, i, 0], [0, 0, 0, -i], [-i, 0, 0, 0], [0, i, 0, 0]], [[0, 0, 1, 0], [0, 0, 0, 1], [1, 0, 0, 0], [0, 1, 0, 0]]]
    return [torch.tensor(m, dtype=torch.complex128, device="cuda") for m in g]


def _wilson(lat, hops, x):
    f, b = hops
    out = torch.zeros_like(x)
    for m, g in enumerate(_gammas()):
        for sign, h in ((-1, _mv(f[m], x[lat.fwd[m]])), (1, _mv(b[m], x[lat.bwd[m]]))):
            out += h + sign * (g[:, :, None] * h[:, None, :, :]).sum(2)
    return out


def _cg(apply, b, tol=1e-13, limit=6000):
    x = torch.zeros_like(b)
    r, p = b.clone(), b.clone()
    rr = b2 = float(torch.linalg.vector_norm(b)) ** 2
    for _ in range(limit):
        if rr <= tol * tol * b2:
            break
        ap = apply(p)
        alpha = rr / float((p.conj() * ap).sum().real)
        x += alpha * p
        r -= alpha * ap
        new = float(torch.linalg.vector_norm(r)) ** 2
        p = r + (new / rr) * p
        rr = new
    return x


def _normal(lat, hops, mass):
    return lambda p: mass * mass * p - _stag(lat, hops, _stag(lat, hops, p))


def _gauge_force(lat, u, beta):
    out = torch.empty_like(u)
    for m in range(4):
        acc = torch.zeros_like(u[:, 0])
        for n in range(4):
            if n != m:
                fm, fn, bn = lat.fwd[m], lat.fwd[n], lat.bwd[n]
                acc += _mm(_mm(u[fm, n], _dag(u[fn, m])), _dag(u[:, n]))
                acc += _mm(_mm(_dag(u[bn[fm], n]), _dag(u[bn, m])), u[bn, n])
        out[:, m] = -(beta / 6.0) * _ta(_mm(u[:, m], acc))
    return out


def _fermion_force(lat, hops, w):
    sign = torch.where(lat.odd, -1.0, 1.0).double()
    out = []
    for m in range(4):
        out.append(_ta(_mv(hops[0][m], w[lat.fwd[m]])[:, :, None] * w.conj()[:, None, :] * sign[:, None, None]))
    return torch.stack(out, 1)


def exact(case, seed):
    inp, d, op = _inputs(case, seed), _dims(case), case["op"]
    lat, u = _Lattice(d), inp["u"]
    hops = _hops(lat, u, op not in ("wilson", "wilson_hop"))
    keep = torch.ones(2, 1, 1, dtype=torch.float64, device="cuda")  # the parities that are written
    if case.get("parity", 2) != 2:
        keep[1 - case["parity"]] = 0
    if op == "dslash":
        b = inp["b"].to(torch.complex64).to(torch.complex128) if case["prec"] else inp["b"]
        return lat.to_eo(_stag(lat, hops, b)) * keep
    if op == "wilson_hop":
        return lat.to_eo(_wilson(lat, hops, inp["b"])) * keep
    if op == "cg":
        x = _cg(_normal(lat, hops, case["mass"]), _keep(lat, inp["b"], case["parity"]))
        out = [lat.to_eo(x)]
        if case.get("y"):
            out.append(lat.to_eo(_stag(lat, hops, x)))
        return out
    if op == "batch":
        return [lat.to_eo(_cg(_normal(lat, hops, m), b)) for b, m in zip(inp["bs"], _masses(case))]
    if op == "serve":
        lat2 = _Lattice(_small(d))
        both = [(lat, hops), (lat2, _hops(lat2, inp["u2"], True))]
        out = []
        for i, (b, m) in enumerate(zip(inp["bs"], _masses(case))):
            la, ho = both[i % 2]
            out.append(la.to_eo(_cg(_normal(la, ho, m), b)))
        return out
    if op == "wilson":
        g5 = torch.tensor([1.0, 1.0, -1.0, -1.0], dtype=torch.float64, device="cuda")[None, :, None]
        mul = lambda p: p - case["kappa"] * _wilson(lat, hops, p)  # noqa: E731
        dag = lambda p: g5 * mul(g5 * p)  # noqa: E731
        return lat.to_eo(_cg(lambda p: dag(mul(p)), dag(inp["b"])))
    if op == "forces":
        return _gauge_force(lat, u, 5.6) + _fermion_force(lat, hops, inp["b"])
    phi = case["mass"] * inp["b"] - _stag(lat, hops, inp["b"])
    phi = _keep(lat, phi, 0)
    q = inp["q"]

    def force(links):
        h = _hops(lat, links, True)
        x = _cg(_normal(lat, h, case["mass"]), phi)
        return _gauge_force(lat, links, 5.6) + _fermion_force(lat, h, x + _stag(lat, h, x))

    eps, n = 0.02, case["steps"]
    q = q + 0.5 * eps * force(u)
    for k in range(n):
        u = _su3(_mm(_exp(eps * q), u))
        q = q + (eps if k < n - 1 else 0.5 * eps) * force(u)
    return [u, q]


def _keep(lat, x, parity):
    """x with the other parity's sites cleared."""
    if parity == 2:
        return x
    return x * (lat.odd == bool(parity))[:, None]
