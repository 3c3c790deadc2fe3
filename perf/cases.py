"""Measured cases: the calls a lattice program makes through the package's public entry points.

The listed cases are the workloads of this repository's tests, benchmark and configurations (the
4^4 operator, 16^4 and 32^4 Wilson hopping, 24^4 x 12 and 16^4 x 16 domain wall, the solvers, the
fermion force, molecular dynamics, multigrid) and one ragged lattice; `draw` spreads more of the
same families over their whole range of extents, precisions, link formats and adjoints.

Inputs are seeded on the device: Haar or weak-field (exp(0.3 i H)) SU(3) links, Gaussian spinors.
`exact` evaluates the operators' definitions in complex128 with plain torch, full 4 x 4 gamma
matrices and full links; the solvers have no such value.
"""
import math

import torch

import paper_1512_03487_amd as gm

DEV = "cuda"

# Parameters of the operators, those of the repository's workloads.
MASS, M5, MF, B5, C5 = 0.1, 1.8, 0.01, 1.5, 0.5
BETA, EPS = 5.6, 0.05   # gauge coupling and step size of the molecular dynamics


def _op(name, kind, dims, ls, prec, links="L18", dag=False, field="haar"):
    return {"name": name, "what": "op", "kind": kind, "lx": dims[0], "ly": dims[1], "lz": dims[2], "lt": dims[3],
            "ls": ls, "prec": prec, "links": links, "dag": dag, "field": field}


def listed():
    return [
        # the smallest configuration: one Wilson D on 4^4 (latency of a single call)
        _op("wilson_4^4_f64", "wilson", (4, 4, 4, 4), 0, "f64"),
        # repeated hopping on the 16^4 weak-field lattice, FP64 (reliable updates, HMC)
        _op("hop_16^4_f64", "hop", (16, 16, 16, 16), 0, "f64", field="weak"),
        # the throughput size of the Wilson workload: the benchmark's headline
        _op("hop_32^4_f32", "hop", (32, 32, 32, 32), 0, "f32"),
        # odd extents no tile or domain divides, compressed links, the adjoint
        _op("wilson_dag_21x15x18x25_f32_l12", "wilson", (21, 15, 18, 25), 0, "f32", "L12", True),
        # the sloppy operator of a mixed-precision Wilson solve
        _op("wilson_32^4_f16s_l12", "wilson", (32, 32, 32, 32), 0, "f16s", "L12"),
        # the five-dimensional operator at the domain-wall throughput size
        _op("dwf_24^4x12_f32", "dwf", (24, 24, 24, 24), 12, "f32"),
        # the normal operator (M, then its adjoint) a sloppy domain-wall iteration applies
        _op("mdagm_24^4x12_f16s", "mdagm", (24, 24, 24, 24), 12, "f16s"),
        # a mixed-precision solve on the Moebius normal equations to 1e-10, recorded iterations
        {"name": "cg_mobius_16^4x16_f32", "what": "cg", "kind": "mobius", "lx": 16, "ly": 16, "lz": 16, "lt": 16,
         "ls": 16, "sloppy": "f32", "links": "L18", "graph": True},
        # an even-odd preconditioned domain-wall solve to 1e-10 with FP16-storage iterations
        {"name": "eo_dwf_16^4x16_f16s", "what": "eo", "kind": "dwf", "lx": 16, "ly": 16, "lz": 16, "lt": 16,
         "ls": 16, "sloppy": "f16s", "links": "L18", "graph": True},
        # the backward pass: adjoint and su(3) link force of the domain-wall operator, FP64 (HMC)
        {"name": "force_dwf_16^4x8_f64", "what": "force", "kind": "dwf", "lx": 16, "ly": 16, "lz": 16, "lt": 16,
         "ls": 8, "prec": "f64", "dag": False},
        # gauge molecular dynamics (gauge force, momentum and link updates)
        {"name": "leapfrog_16^4_f64", "what": "md", "lx": 16, "ly": 16, "lz": 16, "lt": 16, "steps": 4,
         "integrator": "leapfrog"},
        # a multigrid-preconditioned Wilson solve with the basis and coarse operator in hand
        {"name": "mg_24^4_n12", "what": "mg", "lx": 24, "ly": 24, "lz": 24, "lt": 24, "block": 4, "nvec": 12},
    ]


# ------------------------------------------------------------------------------------------------
# Drawn cases
# ------------------------------------------------------------------------------------------------

def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _extents(rng, vol_lo, vol_hi, unit=1):
    """Four extents (multiples of unit, at least 2) of a volume spread over the log of the range."""
    while True:
        v = math.exp(rng.uniform(math.log(vol_lo), math.log(vol_hi)))
        e = [max(max(2, unit), unit * int(round(v ** 0.25 * math.exp(rng.uniform(-0.4, 0.4)) / unit))) for _ in range(4)]
        if vol_lo <= e[0] * e[1] * e[2] * e[3] <= vol_hi:
            return e


def draw(rng):
    what = rng.choice(["op"] * 8 + ["force"] * 2 + ["cg", "eo", "md", "mg"])
    if what == "op":
        kind = rng.choice(["hop", "wilson", "wilson", "dwf", "dwf", "mobius", "mdagm"])
        prec = rng.choice(["f64", "f32", "f32", "f16s", "f16s"])
        ls = 0 if kind in ("hop", "wilson") else rng.choice([4, 6, 8, 10, 12, 16, 24])
        hi = 1 << 20 if ls == 0 else (3 << 20) // ls
        dims = _extents(rng, 256, hi, rng.choice([1, 1, 2, 4]))
        c = _op("", kind, dims, ls, prec, rng.choice(["L18", "L12"]), kind != "mdagm" and rng.random() < 0.5,
                rng.choice(["haar", "weak"]))
    elif what == "force":
        kind = rng.choice(["hop", "wilson", "dwf"])
        ls = rng.choice([4, 6, 8, 12, 16]) if kind == "dwf" else 0
        lx, ly, lz, lt = _extents(rng, 256, 1 << 18 if ls == 0 else (1 << 19) // ls, rng.choice([1, 2, 4]))
        c = {"what": "force", "kind": kind, "lx": lx, "ly": ly, "lz": lz, "lt": lt, "ls": ls,
             "prec": rng.choice(["f64", "f32"]), "dag": rng.random() < 0.5}
    elif what in ("cg", "eo"):
        kind = rng.choice(["wilson", "dwf", "mobius"])
        ls = 0 if kind == "wilson" else rng.choice([4, 6, 8, 12, 16])
        lx, ly, lz, lt = _extents(rng, 256, 1 << 16 if ls == 0 else (1 << 18) // ls, 2)
        c = {"what": what, "kind": kind, "lx": lx, "ly": ly, "lz": lz, "lt": lt, "ls": ls,
             "sloppy": rng.choice(["f64", "f32", "f16s"]), "links": rng.choice(["L18", "L12"]), "graph": rng.random() < 0.7}
    elif what == "md":
        lx, ly, lz, lt = _extents(rng, 256, 1 << 17, rng.choice([1, 2]))
        c = {"what": "md", "lx": lx, "ly": ly, "lz": lz, "lt": lt, "steps": rng.choice([1, 2, 4]),
             "integrator": rng.choice(["leapfrog", "omelyan", "force_gradient"])}
    else:
        block = rng.choice([2, 4])
        lx, ly, lz, lt = _extents(rng, 4096, 1 << 16, block)
        c = {"what": "mg", "lx": lx, "ly": ly, "lz": lz, "lt": lt, "block": block, "nvec": rng.choice([4, 6, 8, 12])}
    c.pop("name", None)
    return c


# ------------------------------------------------------------------------------------------------
# Inputs
# ------------------------------------------------------------------------------------------------

def _gen(seed, part):
    g = torch.Generator(device=DEV)
    g.manual_seed(1000003 * (seed % (1 << 40)) + part)
    return g


def _normal(shape, g):
    return torch.randn(shape, generator=g, device=DEV, dtype=torch.float64)


def _complex(shape, g):
    return torch.view_as_complex(_normal(tuple(shape) + (2,), g) * math.sqrt(0.5))


def _sites(c):
    return (c["lt"], c["lz"], c["ly"], c["lx"])


def _mm(a, b):
    """Products of 3 x 3 matrices."""
    return a[..., :, 0, None] * b[..., None, 0, :] + a[..., :, 1, None] * b[..., None, 1, :] + \
        a[..., :, 2, None] * b[..., None, 2, :]


def _dagger(a):
    return a.conj().transpose(-1, -2)


def _row2(u):
    """Third row of an SU(3) matrix from the first two."""
    r0, r1 = u[..., 0, :], u[..., 1, :]
    r2 = torch.stack([r0[..., 1] * r1[..., 2] - r0[..., 2] * r1[..., 1], r0[..., 2] * r1[..., 0] - r0[..., 0] * r1[..., 2],
                      r0[..., 0] * r1[..., 1] - r0[..., 1] * r1[..., 0]], -1).conj()
    return torch.cat([u[..., :2, :], r2[..., None, :]], -2)


def _unitary(z):
    """SU(3) matrices whose first two rows are z's orthonormalised (Gaussian z: Haar)."""
    r0 = z[..., 0, :] / z[..., 0, :].abs().square().sum(-1, keepdim=True).sqrt()
    r1 = z[..., 1, :] - (r0.conj() * z[..., 1, :]).sum(-1, keepdim=True) * r0
    r1 = r1 / r1.abs().square().sum(-1, keepdim=True).sqrt()
    return _row2(torch.stack([r0, r1], -2))


def _algebra(shape, g):
    """Random su(3) elements i sum_a h_a lambda_a / 2, h_a ~ N(0, 1)."""
    h = _normal(tuple(shape) + (8,), g)
    m = torch.zeros(tuple(shape) + (3, 3), dtype=torch.complex128, device=DEV)
    for k, (i, j) in enumerate(((0, 1), (0, 2), (1, 2))):
        off = torch.complex(h[..., 2 * k], -h[..., 2 * k + 1])
        m[..., i, j] = off
        m[..., j, i] = off.conj()
    d = h[..., 7] / math.sqrt(3.0)
    m[..., 0, 0] = torch.complex(h[..., 6] + d, torch.zeros_like(d))
    m[..., 1, 1] = torch.complex(d - h[..., 6], torch.zeros_like(d))
    m[..., 2, 2] = torch.complex(-2 * d, torch.zeros_like(d))
    return 0.5j * m


def _expm(x, order=18):
    one = torch.eye(3, dtype=torch.complex128, device=DEV)
    e = one.expand(x.shape).clone()
    for n in range(order, 0, -1):
        e = one + _mm(x, e) / n
    return e


def _links(c, seed, kind):
    shape = _sites(c) + (4,)
    if kind == "haar":
        return _unitary(_complex(shape + (3, 3), _gen(seed, 1))).contiguous()
    return _unitary(_expm(0.3 * _algebra(shape, _gen(seed, 1)))).contiguous()


def _spinor(c, seed, part):
    return _complex(_sites(c) + ((c["ls"],) if c.get("ls") else ()) + (4, 3), _gen(seed, part))


def _op_inputs(c, seed):
    """The stored links and spinor of an operator case."""
    u = _links(c, seed, c["field"])
    u = u if c["prec"] == "f64" and c["links"] == "L18" else gm.convert_links(u, c["prec"], c["links"])
    psi = _spinor(c, seed, 2)
    return u, psi if c["prec"] == "f64" else gm.convert_spinor(psi, c["prec"])


def _like(psi):
    return gm.F16Spinor.empty(psi.shape[:-2], psi.device) if isinstance(psi, gm.F16Spinor) else torch.empty_like(psi)


def _bytes(n):
    return torch.empty(n, dtype=torch.uint8, device=DEV)


def _solver_args(c):
    return {"kind": c["kind"], "mass": MASS, "M5": M5, "mf": MF, "b5": B5, "c5": C5, "tol": 1e-10,
            "sloppy": c["sloppy"], "link_fmt": c["links"], "graph": c["graph"]}


_MG = {"setup_rounds": 3, "setup_iters": 20, "coarse_iters": 8, "coarse_tol": 0.25, "smooth_iters": 4, "restart": 8,
       "maxiter": 200, "tol": 1e-10, "setup_prec": "f32", "cycle_prec": "f32"}
_MG_MASS = -0.1


def prepare(case, seed):
    c = case
    if c["what"] == "op":
        u, psi = _op_inputs(c, seed)
        # a program that applies an operator again and again keeps its output (and intermediate)
        return {"c": c, "u": u, "psi": psi, "out": _like(psi), "tmp": _like(psi) if c["kind"] in ("mobius", "mdagm") else None}
    if c["what"] == "force":
        u, psi, g = _links(c, seed, "haar"), _spinor(c, seed, 2), _spinor(c, seed, 3)
        if c["prec"] == "f32":
            u, psi, g = gm.convert_links(u, "f32"), gm.convert_spinor(psi, "f32"), gm.convert_spinor(g, "f32")
        return {"c": c, "u": u, "psi": psi, "g": g}
    if c["what"] in ("cg", "eo"):
        a = _solver_args(c)
        p = {k: a[k] for k in ("tol", "sloppy", "link_fmt", "graph")}
        b = _spinor(c, seed, 2)
        ws = gm.cg_workspace_bytes(b, **p) if c["what"] == "cg" else gm.solve_eo_workspace_bytes(b, **p)
        return {"c": c, "u": _links(c, seed, "haar"), "b": b, "args": a, "ws": _bytes(ws)}
    if c["what"] == "md":
        u, p = _links(c, seed, "weak"), _algebra(_sites(c) + (4,), _gen(seed, 4))
        return {"c": c, "u": u, "p": p, "u1": torch.empty_like(u), "p1": torch.empty_like(p)}
    u, b = _links(c, seed, "weak"), _spinor(c, seed, 2)
    vecs = _complex((c["nvec"],) + _sites(c) + (4, 3), _gen(seed, 5))
    par = dict(_MG, block=(c["block"],) * 4)
    ws = _bytes(gm.mg_workspace_bytes(u, nvec=c["nvec"], **par))
    gm.mg_basis(u, vecs, _MG_MASS, workspace=ws, **par)
    a = gm.mg_coarse_op(u, vecs, _MG_MASS, workspace=ws, **par)
    return {"c": c, "u": u, "b": b, "vecs": vecs, "a": a, "par": par, "ws": ws}


def _plain(x):
    return {"codes": x.codes, "scale": x.scale} if isinstance(x, gm.F16Spinor) else x


def run(state):
    s, c = state, state["c"]
    if c["what"] == "op":
        k, dag = c["kind"], c["dag"]
        if k == "hop":
            return _plain(gm.dhop(s["u"], s["psi"], "hop", dag=dag, out=s["out"]))
        if k == "wilson":
            return _plain(gm.wilson(s["u"], s["psi"], MASS, dag=dag, out=s["out"]))
        if k == "dwf":
            return _plain(gm.dwf(s["u"], s["psi"], M5, MF, dag=dag, out=s["out"]))
        if k == "mobius":
            return _plain(gm.mobius(s["u"], s["psi"], M5, MF, B5, C5, dag=dag, out=s["out"], tmp=s["tmp"]))
        return _plain(gm.dwf_mdag_m(s["u"], s["psi"], M5, MF, out=s["out"], tmp=s["tmp"]))
    if c["what"] == "force":
        gp, gu = gm.dhop_backward(s["u"], s["psi"], s["g"], c["kind"], dag=c["dag"], mass=MASS, M5=M5, mf=MF, force=True)
        return {"psi": gp, "u": gu}
    if c["what"] == "cg":
        return gm.cg(s["u"], s["b"], workspace=s["ws"], **s["args"])[0]
    if c["what"] == "eo":
        return gm.solve_eo(s["u"], s["b"], workspace=s["ws"], **s["args"])[0]
    if c["what"] == "md":
        # a trajectory keeps its starting configuration for the Metropolis test
        u, p = s["u1"].copy_(s["u"]), s["p1"].copy_(s["p"])
        gm.md_leapfrog(u, p, BETA, EPS, c["steps"], integrator=c["integrator"])
        return {"u": u, "p": p}
    return gm.mg_solve(s["u"], s["vecs"], s["a"], s["b"], _MG_MASS, workspace=s["ws"], **s["par"])[0]


# ------------------------------------------------------------------------------------------------
# Work
# ------------------------------------------------------------------------------------------------

_SPINOR = {"f64": 192, "f32": 96, "f16s": 52}
_REAL = {"f64": 8, "f32": 4, "f16s": 2}


def _apply_work(vol, ls, prec, links, kind):
    """One application: psi, out and the four links of each site once; 1320 flops per 5D site for the
    hopping term, 48 for a Wilson diagonal, 96 for a fifth dimension."""
    n5 = vol * max(1, ls)
    b = 2 * n5 * _SPINOR[prec] + vol * 4 * (18 if links == "L18" else 12) * _REAL[prec]
    extra = {"hop": 0, "wilson": 48, "dwf": 96, "mobius": 288}[kind]
    return b, n5 * (1320 + extra)


def work(case):
    c = case
    vol = c["lx"] * c["ly"] * c["lz"] * c["lt"]
    ls = c.get("ls", 0)
    n5 = vol * max(1, ls)
    if c["what"] == "op":
        two = c["kind"] == "mdagm"
        b, f = _apply_work(vol, ls, c["prec"], c["links"], "dwf" if two else c["kind"])
        return {"bytes": 2 * b if two else b, "flops": 2 * f if two else f}
    if c["what"] == "force":
        # the adjoint, then psi, g and the links read and the force written
        b, f = _apply_work(vol, ls, c["prec"], "L18", c["kind"])
        sp, lk = n5 * _SPINOR[c["prec"]], vol * 4 * 18 * _REAL[c["prec"]]
        return {"bytes": b + 2 * sp + 2 * lk, "flops": f + vol * 4 * 400 + n5 * 4 * 336}
    if c["what"] in ("cg", "eo"):
        # a nominal iteration count; per iteration two applications and x, p, r read, x, p written
        its = {"wilson": 60, "dwf": 530, "mobius": 500}[c["kind"]] if c["what"] == "cg" else {"wilson": 30, "dwf": 210, "mobius": 270}[c["kind"]]
        b, f = _apply_work(vol, ls, c["sloppy"], c["links"], c["kind"])
        part = 1.0 if c["what"] == "cg" else 0.5
        vec = 3 * _SPINOR[c["sloppy"]] + 2 * (192 if c["sloppy"] == "f64" else 96)
        return {"bytes": its * (2 * b + part * n5 * vec), "flops": its * (2 * f + part * n5 * 200)}
    if c["what"] == "md":
        per = {"leapfrog": (1, 1), "omelyan": (2, 2), "force_gradient": (3, 3)}[c["integrator"]]
        lb = vol * 4 * 144
        # a force reads U and updates P (read, write); a link update reads P and updates U
        return {"bytes": 3 * lb * ((per[0] * c["steps"] + 1) + per[1] * c["steps"]) + 4 * lb,
                "flops": vol * 4 * (2900 * (per[0] * c["steps"] + 1) + 3800 * per[1] * c["steps"])}
    # multigrid: a nominal 35 cycles, each with one FP64 and five FP32 applications, the FP32 basis
    # read for restriction and prolongation and 16 coarse stencils with FP32 matrices
    b, f = _apply_work(vol, 0, "f64", "L18", "wilson")
    vc, n = vol // c["block"] ** 4, 2 * c["nvec"]
    coarse = vc * 9 * n * n
    return {"bytes": 35 * (b + 5 * b / 2 + 2 * c["nvec"] * vol * 96 + 16 * coarse * 8),
            "flops": 35 * (6 * f + 2 * c["nvec"] * vol * 96 + 16 * coarse * 8)}


# ------------------------------------------------------------------------------------------------
# The definitions in complex128
# ------------------------------------------------------------------------------------------------

def _gammas():
    s = torch.tensor([[[0, 1], [1, 0]], [[0, -1j], [1j, 0]], [[1, 0], [0, -1]]], dtype=torch.complex128, device=DEV)
    g = torch.zeros(4, 4, 4, dtype=torch.complex128, device=DEV)
    for k in range(3):
        g[k, :2, 2:], g[k, 2:, :2] = -1j * s[k], 1j * s[k]
    g[3, :2, 2:] = g[3, 2:, :2] = torch.eye(2, dtype=torch.complex128, device=DEV)
    return g


def _spin(m, p):
    """m acting on the spin index (the last but one)."""
    return torch.stack([sum(m[a, b] * p[..., b, :] for b in range(4) if m[a, b] != 0) for a in range(4)], -2)


def _colour(u, p):
    return sum(u[..., None, :, b] * p[..., :, b, None] for b in range(3))


def _hop4(u, p, dag):
    """H psi of a 4D field: forward 1 - gamma, backward 1 + gamma (exchanged for the adjoint)."""
    g, one, e = _gammas(), torch.eye(4, dtype=torch.complex128, device=DEV), 1.0 if dag else -1.0
    out = torch.zeros_like(p)
    for mu in range(4):
        d = 3 - mu
        out += _spin(one + e * g[mu], _colour(u[..., mu, :, :], p.roll(-1, d)))
        out += _spin(one - e * g[mu], _colour(_dagger(u[..., mu, :, :]), p).roll(1, d))
    return out


def _hop(u, p, dag):
    if p.dim() == 6:
        return _hop4(u, p, dag)
    out = torch.empty_like(p)
    for s in range(p.shape[4]):
        out[:, :, :, :, s] = _hop4(u, p[:, :, :, :, s], dag)
    return out


def _shift5(p, dag):
    """S psi: the lower spins from s + 1, the upper from s - 1, -mf across the wall (exchanged for S^+)."""
    up, dn = p.roll(-1, 4), p.roll(1, 4)
    up[:, :, :, :, -1] *= -MF
    dn[:, :, :, :, 0] *= -MF
    if dag:
        up, dn = dn, up
    return torch.cat([dn[..., :2, :], up[..., 2:, :]], -2)


def _apply(u, p, kind, dag):
    if kind == "hop":
        return _hop(u, p, dag)
    if kind == "wilson":
        return (4.0 + MASS) * p - 0.5 * _hop(u, p, dag)
    if kind == "dwf":
        return (5.0 - M5) * p - 0.5 * _hop(u, p, dag) - _shift5(p, dag)
    if not dag:
        q = B5 * p + C5 * _shift5(p, False)
        return (4.0 - M5) * q - 0.5 * _hop(u, q, False) + p - _shift5(p, False)
    q = (4.0 - M5) * p - 0.5 * _hop(u, p, True)
    return B5 * q + C5 * _shift5(q, True) + p - _shift5(p, True)


def _wide(u, psi):
    """The stored values in complex128, the third row of compressed links rebuilt."""
    if u.dtype == torch.float16:
        u = torch.view_as_complex(u.double())
    u = u.to(torch.complex128)
    if u.shape[-2] == 2:
        u = _row2(u)
    if isinstance(psi, gm.F16Spinor):
        return u, torch.view_as_complex((psi.codes.float() * psi.scale[..., None, None, None]).double())
    return u, psi.to(torch.complex128)


def _coded(out, prec):
    if prec != "f16s":
        return out
    v = torch.view_as_real(out)
    m = v.abs().amax((-3, -2, -1))
    return {"codes": v / m[..., None, None, None], "scale": m}


def _ta(a):
    """Traceless anti-Hermitian part."""
    m = 0.5 * (a - _dagger(a))
    t = (m[..., 0, 0] + m[..., 1, 1] + m[..., 2, 2]) / 3.0
    return m - t[..., None, None] * torch.eye(3, dtype=torch.complex128, device=DEV)


def _outer(a, b):
    """sum over spin (and s) of a b^+ as colour matrices."""
    a, b = (x if x.dim() == 7 else x[:, :, :, :, None] for x in (a, b))
    out = 0
    for s in range(a.shape[4]):
        for k in range(4):
            out = out + a[:, :, :, :, s, k, :, None] * b[:, :, :, :, s, k, None, :].conj()
    return out


def _force(u, psi, chi, kind, dag):
    g, one, e = _gammas(), torch.eye(4, dtype=torch.complex128, device=DEV), 1.0 if dag else -1.0
    out = torch.empty_like(u)
    for mu in range(4):
        d = 3 - mu
        grad = _outer(_spin(one + e * g[mu], chi), psi.roll(-1, d)) + _outer(psi, _spin(one - e * g[mu], chi.roll(-1, d)))
        out[..., mu, :, :] = _ta((1.0 if kind == "hop" else -0.5) * _mm(grad, _dagger(u[..., mu, :, :])))
    return out


def _gauge_force(u):
    f = torch.empty_like(u)
    for mu in range(4):
        st = 0
        um = u[..., mu, :, :]
        for nu in range(4):
            if nu == mu:
                continue
            un = u[..., nu, :, :]
            st = st + _mm(_mm(un.roll(-1, 3 - mu), _dagger(um.roll(-1, 3 - nu))), _dagger(un))
            low = _mm(_mm(_dagger(un.roll(-1, 3 - mu)), _dagger(um)), un)
            st = st + low.roll(1, 3 - nu)
        f[..., mu, :, :] = (BETA / 3.0) * _ta(_mm(um, st))
    return f


def _leapfrog(u, p, steps):
    p = p - 0.25 * EPS * _gauge_force(u)
    for k in range(steps):
        u = _mm(_expm(EPS * p), u)
        p = p - (0.5 if k + 1 < steps else 0.25) * EPS * _gauge_force(u)
    return {"u": u, "p": p}


def exact(case, seed):
    c = case
    if c["what"] == "op":
        u, psi = _wide(*_op_inputs(c, seed))
        if c["kind"] == "mdagm":
            return _coded(_apply(u, _apply(u, psi, "dwf", False), "dwf", True), c["prec"])
        return _coded(_apply(u, psi, c["kind"], c["dag"]), c["prec"])
    if c["what"] == "force":
        s = prepare(c, seed)
        u, psi = _wide(s["u"], s["psi"])
        g = s["g"].to(torch.complex128)
        return {"psi": _apply(u, g, c["kind"], not c["dag"]), "u": _force(u, psi, g, c["kind"], c["dag"])}
    if c["what"] == "md" and c["integrator"] == "leapfrog":
        s = prepare(c, seed)
        return _leapfrog(s["u"], s["p"], c["steps"])
    return None
