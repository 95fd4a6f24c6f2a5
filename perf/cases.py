"""The workloads that the library's speed is measured on: what a lattice program has it do.

listed() names them, draw() gives more of the same ranges, prepare() makes what the program
holds before the call (links, fields, packed gauge fields, solver workspaces), run() is one
call (or one short chain of calls) through the package's entry points, work() the bytes and
operations that the call cannot do without, and exact() the same result in plain torch with
64-bit arithmetic, from the definitions alone.

Kinds of work, and their ranges:

  operator   D_eo, D_oe and the normal operator m^2 - D_eo D_oe: 4^4 to 32^4 sites, all four
             link formats, 1 to 12 fields, standard or stored phases
  cg         cg_solve: 4^4 to 32^4, FP64 or mixed precision, 1 to 8 right-hand sides
  shifted    multishift_cg_solve and rational_apply: 6^4 to 24^3 x 48, 4 to 16 poles
  batch      cg_solve_batch: up to some twenty solves on lattices of 4^4 to 16^4
  staples    gauge_staples: 4^4 to 32^4, all four link formats
  md         one pure-gauge molecular-dynamics step (momentum, then link update)
  force      the smeared fermion force: one stout level, the force of the rational action on
             the smeared links, and its chain down to the thin links
"""
from __future__ import annotations

import math

import torch

import paper_1701_00426_amd as stg

FORMATS = ("c128_18", "c128_12", "c64_12", "bf16_12")
LINK_BYTES = {"c128_18": 144, "c128_12": 96, "c64_12": 48, "bf16_12": 24}  # one link


def listed():
    return [
        # the smallest call: one hop of one field on a lattice that does not fill the chip
        {"name": "hop_8_f64", "kind": "operator", "op": "oe", "dims": "8 8 8 8",
         "fmt": "c128_18", "nrhs": 1, "phases": False},
        # the benchmark's hop
        {"name": "hop_32_f64", "kind": "operator", "op": "eo", "dims": "32 32 32 32",
         "fmt": "c128_12", "nrhs": 1, "phases": False},
        # the operator of a solve with several right-hand sides
        {"name": "normal_32_f32_8", "kind": "operator", "op": "normal", "dims": "32 32 32 32",
         "fmt": "c64_12", "nrhs": 8, "phases": False},
        # uneven extents, BF16 links, the program's own phases (e.g. with a chemical potential)
        {"name": "normal_uneven_bf16_3", "kind": "operator", "op": "normal",
         "dims": "20 12 18 28", "fmt": "bf16_12", "nrhs": 3, "phases": True},
        # a small solve, all latency
        {"name": "cg_8_f64", "kind": "cg", "dims": "8 8 8 8", "mass": 0.1, "nrhs": 1,
         "hi": "c128_18", "lo": ""},
        # the benchmark's solve: mixed precision at a light mass
        {"name": "cg_32_mixed", "kind": "cg", "dims": "32 32 32 32", "mass": 0.01, "nrhs": 1,
         "hi": "c128_12", "lo": "c64_12"},
        # the solve of an RHMC force: every pole at once, two pseudofermions
        {"name": "multishift_24x48_mixed", "kind": "shifted", "op": "multishift",
         "dims": "24 24 24 48", "mass": 0.02, "nrhs": 2, "poles": 16, "hi": "c128_12",
         "lo": "c64_12"},
        # the heat bath of a smaller lattice: a rational function to full precision
        {"name": "rational_16x32_f64", "kind": "shifted", "op": "rational",
         "dims": "16 16 16 32", "mass": 0.05, "nrhs": 4, "poles": 10, "hi": "c128_12",
         "lo": ""},
        # many small solves of an ensemble study, advanced together
        {"name": "batch_small_mixed", "kind": "batch", "solves": 16, "smallest": 8,
         "largest": 16, "mass": 0.05, "hi": "c128_12", "lo": "c64_12"},
        # single-precision staples (the gauge force of a single-precision trajectory)
        {"name": "staples_24_f32", "kind": "staples", "dims": "24 24 24 24", "fmt": "c64_12"},
        # one pure-gauge step of a trajectory
        {"name": "md_32_f64", "kind": "md", "dims": "32 32 32 32", "fmt": "c128_12"},
        # the fermion force of a stout-smeared action
        {"name": "smeared_force_24x48", "kind": "force", "dims": "24 24 24 48", "poles": 12,
         "fmt": "c128_12"},
    ]


def _draw_dims(rng, lo, hi):
    """Even extents, volume spread over the logarithm of [lo, hi], unequal as a rule."""
    while True:
        side = (lo * (hi / lo) ** rng.random()) ** 0.25
        dims = [max(2, 2 * round(side * rng.uniform(0.6, 1.6) / 2)) for _ in range(4)]
        if lo <= math.prod(dims) <= hi:
            return " ".join(map(str, dims))


def draw(rng):
    kind = rng.choice(("operator", "operator", "cg", "shifted", "batch", "staples", "md", "force"))
    if kind == "operator":
        return {"kind": kind, "op": rng.choice(("eo", "oe", "normal")),
                "dims": _draw_dims(rng, 4**4, 32**4), "fmt": rng.choice(FORMATS),
                "nrhs": rng.choice((1, 1, 2, 3, 4, 6, 8, 12)), "phases": rng.random() < 0.3}
    if kind == "cg":
        lo = rng.choice(("", "c64_12", "c64_12", "bf16_12"))
        return {"kind": kind, "dims": _draw_dims(rng, 4**4, 20**4),
                "mass": round(math.exp(rng.uniform(math.log(0.02), math.log(0.2))), 3),
                "nrhs": rng.choice((1, 1, 1, 2, 4, 8)), "hi": rng.choice(("c128_12", "c128_18")),
                "lo": lo}
    if kind == "shifted":
        return {"kind": kind, "op": rng.choice(("multishift", "rational")),
                "dims": _draw_dims(rng, 6**4, 20**4),
                "mass": round(math.exp(rng.uniform(math.log(0.02), math.log(0.1))), 3),
                "nrhs": rng.choice((1, 1, 2, 3, 8)), "poles": rng.randint(4, 16),
                "hi": "c128_12", "lo": rng.choice(("", "c64_12", "c64_12"))}
    if kind == "batch":
        return {"kind": kind, "solves": rng.randint(3, 20), "smallest": rng.choice((4, 6, 8)),
                "largest": rng.choice((8, 12, 16)), "mass": round(rng.uniform(0.04, 0.2), 3),
                "hi": "c128_12", "lo": rng.choice(("", "c64_12", "c64_12"))}
    if kind == "staples":
        return {"kind": kind, "dims": _draw_dims(rng, 4**4, 32**4), "fmt": rng.choice(FORMATS)}
    if kind == "md":
        return {"kind": kind, "dims": _draw_dims(rng, 4**4, 32**4), "fmt": rng.choice(FORMATS[:3])}
    return {"kind": kind, "dims": _draw_dims(rng, 4**4, 20**4), "poles": rng.randint(3, 20),
            "fmt": rng.choice(FORMATS[:2])}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
RHO = 0.15                       # stout weight
BETA, EPS = 5.5, 0.01            # gauge coupling and step of the molecular dynamics
TOL = 1e-10                      # stopping test of every solve


def _dims(case):
    return tuple(int(n) for n in case["dims"].split())


def _half(dims):
    return math.prod(dims) // 2


def _gen(seed, part):
    g = torch.Generator("cuda")
    g.manual_seed((int(seed) * 64 + part) % (1 << 60))
    return g


def _normal(g, *shape):
    z = torch.randn(*shape, 2, generator=g, device="cuda", dtype=torch.float64)
    return torch.view_as_complex(z)


def _links(dims, seed, part=0):
    """Random SU(3) links (8, 3, 3, Vh): two Gaussian rows, orthonormalised, third their
    conjugate cross product (as seeded_inputs does on the host)."""
    g = _gen(seed, part)
    a = _normal(g, 8, 3, _half(dims))
    a /= a.abs().square().sum(1, keepdim=True).sqrt()
    b = _normal(g, 8, 3, _half(dims))
    b -= (a.conj() * b).sum(1, keepdim=True) * a
    b /= b.abs().square().sum(1, keepdim=True).sqrt()
    return torch.stack([a, b, torch.linalg.cross(a, b, dim=1).conj()], 1).contiguous()


def _momenta(dims, seed):
    """Traceless Hermitian Gaussian momenta (8, 3, 3, Vh)."""
    a = _normal(_gen(seed, 3), 8, 3, 3, _half(dims))
    h = 0.5 * (a + a.transpose(1, 2).conj())
    tr = (h[:, 0, 0] + h[:, 1, 1] + h[:, 2, 2]) / 3
    for i in range(3):
        h[:, i, i] -= tr
    return h.contiguous()


def _phases(dims, seed):
    """Real phases (8, Vh) that a program brings along."""
    u = torch.rand(8, _half(dims), generator=_gen(seed, 2), device="cuda", dtype=torch.float64)
    return 2 * u - 1


def _shifts(case):
    n, lo, hi = case["poles"], 1e-4, 10.0
    return [lo * (hi / lo) ** (k / (n - 1)) for k in range(n)]


def _weights(case):
    return [0.05 * s ** 0.5 for s in _shifts(case)]


def _batch_plan(case):
    """(dims, nrhs, mass) of each solve of a batch: extents between the two sides given."""
    lo, hi = sorted((case["smallest"], case["largest"]))
    sides = list(range(lo, hi + 1, 2))
    plan = []
    for i in range(case["solves"]):
        n, t = sides[(5 * i) % len(sides)], sides[(3 * i + 1) % len(sides)]
        plan.append(((n, n, n, t), 1 + i % 4, case["mass"] * (1 + i % 2)))
    return plan


def _field_dtype(fmt):
    return torch.complex128 if fmt.startswith("c128") else torch.complex64


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        solves = []
        for i, (dims, nrhs, mass) in enumerate(_batch_plan(case)):
            links = _links(dims, seed, 8 + i)
            sv = {"hi": stg.pack_gauge(dims, links, case["hi"]), "mass": mass,
                  "b": _normal(_gen(seed, 36 + i), nrhs, 3, _half(dims))}
            if case["lo"]:
                sv["lo"] = stg.pack_gauge(dims, links, case["lo"])
            solves.append(sv)
        return {"case": case, "solves": solves}
    dims = _dims(case)
    links = _links(dims, seed)
    state = {"case": case}
    if kind == "operator":
        state["gauge"] = stg.pack_gauge(dims, links, case["fmt"],
                                        _phases(dims, seed) if case["phases"] else None)
        dt = _field_dtype(case["fmt"])
        state["in"] = _normal(_gen(seed, 1), case["nrhs"], 3, _half(dims)).to(dt)
        state["out"] = torch.empty_like(state["in"])
        state["tmp"] = torch.empty_like(state["in"])
    elif kind in ("cg", "shifted"):
        state["hi"] = stg.pack_gauge(dims, links, case["hi"])
        state["lo"] = stg.pack_gauge(dims, links, case["lo"]) if case["lo"] else None
        state["b"] = _normal(_gen(seed, 1), case["nrhs"], 3, _half(dims))
        mode = stg.STG_CG_MIXED if case["lo"] else stg.STG_CG_F64
        if kind == "cg":
            size = stg.stg_workspace_bytes(dims, case["nrhs"], 0, mode)
        elif case["op"] == "multishift":
            size = stg.stg_workspace_bytes(dims, case["nrhs"], case["poles"], mode)
        else:
            size = stg.stg_rational_workspace_bytes(dims, case["nrhs"], case["poles"], mode)
        state["ws"] = torch.empty(size, dtype=torch.uint8, device="cuda")
    elif kind == "staples":
        state["gauge"] = stg.pack_gauge(dims, links, case["fmt"])
        state["out"] = torch.empty((8, 3, 3, _half(dims)), dtype=_field_dtype(case["fmt"]),
                                   device="cuda")
    elif kind == "md":
        state["gauge"] = stg.pack_gauge(dims, links, case["fmt"])
        state["mom"] = _momenta(dims, seed).to(_field_dtype(case["fmt"]))
    else:
        state["thin"] = stg.pack_gauge(dims, links, case["fmt"])
        state["x"] = _solutions(case, dims, seed)
        for name in ("smeared", "g", "sigma", "ws"):
            state[name] = torch.empty_like(links)
        state["y"] = torch.empty_like(state["x"])
    return state


def _solutions(case, dims, seed):
    """Fields with the norms that the solutions of the shifted systems have."""
    x = _normal(_gen(seed, 1), case["poles"], 3, _half(dims))
    return x / torch.tensor([1.0 + s for s in _shifts(case)], device="cuda")[:, None, None]


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "operator":
        if case["op"] == "normal":
            return stg.stg_apply_normal(state["gauge"], 0.05, state["in"], out_even=state["out"],
                                        tmp_odd=state["tmp"])
        apply = stg.dirac_apply_eo if case["op"] == "eo" else stg.dirac_apply_oe
        return apply(state["gauge"], state["in"], state["out"])
    if kind == "cg":
        return stg.cg_solve(state["hi"], case["mass"], state["b"], lo=state["lo"], ws=state["ws"],
                            tol=TOL)[0]
    if kind == "shifted" and case["op"] == "multishift":
        return stg.multishift_cg_solve(state["hi"], case["mass"], _shifts(case), state["b"],
                                       lo=state["lo"], ws=state["ws"], tol=TOL)[0]
    if kind == "shifted":
        return stg.rational_apply(state["hi"], case["mass"], _shifts(case), _weights(case), 0.3,
                                  state["b"], lo=state["lo"], ws=state["ws"], tol=TOL)[0]
    if kind == "batch":
        return stg.cg_solve_batch(state["solves"], tol=TOL)[0]
    if kind == "staples":
        return stg.gauge_staples(state["gauge"], out=state["out"])
    if kind == "md":
        gauge, mom = state["gauge"], state["mom"]
        stg.gauge_momentum_update(gauge, mom, BETA, EPS)
        stg.gauge_link_update(gauge, mom, EPS)
        # the packed links are a byte buffer: hand them back as the numbers they hold
        return [gauge.links.view(mom.real.dtype).reshape(-1), mom]
    smeared = stg.stout_smear(state["thin"], RHO, out=state["smeared"])
    gauge = stg.pack_gauge(_dims(case), smeared, "c128_12")
    g, y = stg.fermion_force(gauge, _weights(case), state["x"], state["y"], state["g"])
    sigma = stg.stout_force_backprop(state["thin"], RHO, g, state["sigma"], state["ws"])
    return [smeared, y, g, sigma]


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
HOP_FLOPS = 570.0                # per output site and field


def _solve_work(dims, fmt, nrhs, light, elem):
    """Iterations (about 31 / sqrt(m^2 + smallest shift) on random links) of one operator
    application, the links read once, and x, r and p of every field read and written once."""
    vh, iters = _half(dims), 31.0 / light
    return {"bytes": iters * vh * (8 * LINK_BYTES[fmt] + 6 * 3 * elem * nrhs),
            "flops": iters * vh * nrhs * 2 * HOP_FLOPS}


def work(case):
    kind = case["kind"]
    if kind == "batch":
        fmt = case["lo"] or case["hi"]
        each = [_solve_work(dims, fmt, nrhs, mass, 8 if case["lo"] else 16)
                for dims, nrhs, mass in _batch_plan(case)]
        return {k: sum(w[k] for w in each) for k in ("bytes", "flops")}
    vh = _half(_dims(case))
    if kind == "operator":
        elem = 16 if case["fmt"].startswith("c128") else 8
        hops = 2 if case["op"] == "normal" else 1
        return {"bytes": vh * (8 * LINK_BYTES[case["fmt"]] + (4 * elem if case["phases"] else 0)
                               + 2 * 3 * elem * case["nrhs"]),
                "flops": HOP_FLOPS * hops * vh * case["nrhs"]}
    if kind in ("cg", "shifted"):
        fmt, elem = case["lo"] or case["hi"], 8 if case["lo"] else 16
        light = case["mass"]
        if kind == "shifted":
            light = math.sqrt(light * light + _shifts(case)[0])
        w = _solve_work(_dims(case), fmt, case["nrhs"], light, elem)
        if kind == "shifted":    # and the solution of every pole, written once
            w["bytes"] += vh * 48.0 * case["nrhs"] * case["poles"]
        return w
    elem = 16 if case["fmt"].startswith("c128") else 8
    link = LINK_BYTES[case["fmt"]]
    if kind == "staples":
        return {"bytes": 8.0 * vh * (link + 9 * elem), "flops": 8.0 * vh * 13824}
    if kind == "md":
        return {"bytes": 8.0 * vh * (2 * link + 2 * 9 * elem), "flops": 8.0 * vh * (13824 + 1600)}
    return {"bytes": 8.0 * vh * (link + 3 * 144) + 2.0 * vh * 48 * case["poles"],
            "flops": vh * (8 * (3375.0 + 21500.0) + case["poles"] * (HOP_FLOPS + 8 * 72))}


# ---------------------------------------------------------------------------
# the same results from the definitions, in 64 bits
# ---------------------------------------------------------------------------
class _Lattice:
    """Index tables of the even/odd layout: sites of one parity in half-lexicographic order."""

    def __init__(self, dims):
        self.dims = dims
        n0, n1, n2, n3 = dims
        h = torch.arange(_half(dims), device="cuda")
        rest = h // (n0 // 2)
        x1, x2, x3 = rest % n1, rest // n1 % n2, rest // (n1 * n2)
        self.x = []              # coordinates of the sites of each parity
        for par in (0, 1):
            x0 = 2 * (h % (n0 // 2)) + (x1 + x2 + x3 + par) % 2
            self.x.append([x0, x1, x2, x3])

    def near(self, par, mu, step):
        """Half index of x + step mu for the sites x of parity par."""
        x = list(self.x[par])
        x[mu] = (x[mu] + step) % self.dims[mu]
        n0, n1, n2, _ = self.dims
        return (x[0] + n0 * (x[1] + n1 * (x[2] + n2 * x[3]))) // 2

    def phases(self):
        """Standard staggered phases (8, Vh), antiperiodic in the last direction."""
        out = []
        for mu in range(4):
            for par in (0, 1):
                x = self.x[par]
                s = 1 - 2 * (sum(x[:mu], torch.zeros_like(x[0])) % 2)
                if mu == 3:
                    s = torch.where(x[3] == self.dims[3] - 1, -s, s)
                out.append(s.double())
        return torch.stack(out)


def _dag(a):
    return a.transpose(0, 1).conj()


def _mul(a, b):
    """Product of two fields of 3x3 matrices (3, 3, n)."""
    return a[:, 0, None] * b[None, 0] + a[:, 1, None] * b[None, 1] + a[:, 2, None] * b[None, 2]


def _stored(links, fmt):
    """The links as the format keeps them: rounded, the third row rebuilt."""
    if fmt == "c128_18":
        return links
    rows = torch.view_as_real(links[:, :2].contiguous())
    if fmt == "c64_12":
        rows = rows.float().double()
    elif fmt == "bf16_12":
        # 8 significant bits, to nearest even, straight from the double
        m, e = torch.frexp(rows)
        rows = torch.ldexp(torch.round(m * 256.0) / 256.0, e)
    rows = torch.view_as_complex(rows.contiguous())
    third = torch.linalg.cross(rows[:, 0], rows[:, 1], dim=1).conj()
    return torch.cat([rows, third[:, None]], 1)


class _Operator:
    """D_eo and D_oe with links and phases folded into one matrix per site and direction."""

    def __init__(self, dims, links, phases=None):
        lat = _Lattice(dims)
        ph = lat.phases() if phases is None else phases
        self.m, self.at = [], []
        for par in (0, 1):
            m, at = [], []
            for mu in range(4):
                s, o = 2 * mu + par, 2 * mu + 1 - par
                back = lat.near(par, mu, -1)
                m += [0.5 * ph[s] * links[s], -0.5 * (ph[o] * _dag(links[o]))[..., back]]
                at += [lat.near(par, mu, 1), back]
            self.m.append(torch.stack(m))
            self.at.append(torch.stack(at))

    def hop(self, par, v):
        """Fields (n, 3, Vh) on the other parity to those on parity par."""
        out = torch.empty_like(v)
        for j in range(v.shape[0]):
            g = v[j][:, self.at[par]]                     # (3, 8, Vh)
            out[j] = sum((self.m[par][:, :, b] * g[b][:, None]).sum(0) for b in range(3))
        return out

    def normal(self, diag, v):
        return diag * v - self.hop(0, self.hop(1, v))


def _dots(a, b):
    return (a.conj() * b).real.sum((1, 2))


def _solve(op, diag, b, shifts=(0.0,)):
    """Multi-shift CG in 64 bits, run past the library's tolerance; (shifts, n, 3, Vh)."""
    base = min(shifts)
    d = torch.tensor([s - base for s in shifts], dtype=torch.float64, device=b.device)[:, None]
    x = torch.zeros((len(shifts),) + tuple(b.shape), dtype=b.dtype, device=b.device)
    ps = b.expand(x.shape).clone()
    r, p = b.clone(), b.clone()
    rr = bb = _dots(r, r)
    zeta = zeta0 = torch.ones((len(shifts), b.shape[0]), dtype=torch.float64, device=b.device)
    alpha0, beta0 = torch.ones_like(bb), torch.zeros_like(bb)
    for _ in range(20000):
        q = op.normal(diag + base, p)
        alpha = rr / _dots(p, q)
        den = alpha * beta0 * (zeta0 - zeta) + zeta0 * alpha0 * (1 + d * alpha)
        zeta1 = torch.where(zeta.abs() > 1e-100, zeta * zeta0 * alpha0 / den, 0.0)
        ratio = torch.where(zeta.abs() > 1e-100, zeta1 / zeta, 0.0)
        r -= alpha[:, None, None] * q
        new = _dots(r, r)
        beta = new / rr
        for k in range(len(shifts)):
            x[k] += (alpha * ratio[k])[:, None, None] * ps[k]
            ps[k] *= (beta * ratio[k] ** 2)[:, None, None]
            ps[k] += zeta1[k][:, None, None] * r
        p = r + beta[:, None, None] * p
        zeta0, zeta, alpha0, beta0, rr = zeta, zeta1, alpha, beta, new
        if bool((rr <= 1e-25 * bb).all()):
            return x
    return None


def _full(lat, links):
    """Links by direction on the whole lattice: (4, 3, 3, N3, N2, N1, N0)."""
    n0, n1, n2, n3 = lat.dims
    out = torch.empty((4, 3, 3, n0 * n1 * n2 * n3), dtype=links.dtype, device=links.device)
    for mu in range(4):
        for par in (0, 1):
            x = lat.x[par]
            out[mu][..., x[0] + n0 * (x[1] + n1 * (x[2] + n2 * x[3]))] = links[2 * mu + par]
    return out.reshape(4, 3, 3, n3, n2, n1, n0)


def _slots(lat, full):
    """The inverse of _full."""
    n0, n1, n2, _ = lat.dims
    flat = full.reshape(4, 3, 3, -1)
    return torch.stack([flat[mu][..., x[0] + n0 * (x[1] + n1 * (x[2] + n2 * x[3]))]
                        for mu in range(4) for x in lat.x])


def _at(f, *moves):
    """The field seen from x + sum of moves (mu, step)."""
    for mu, step in moves:
        f = torch.roll(f, -step, dims=f.dim() - 1 - mu)
    return f


def _line(u, path):
    """Product of the links met along a path of signed directions (+-(mu + 1)) from x."""
    here, prod = [], None
    for step in path:
        mu = abs(step) - 1
        if step > 0:
            link = _at(u[mu], *here)
            here.append((mu, 1))
        else:
            here.append((mu, -1))
            link = _dag(_at(u[mu], *here))
        prod = link if prod is None else _mul(prod, link)
    return prod


def _staple(u, mu, c0, c1):
    """Sum over the 3- and 5-link paths from x + mu back to x."""
    f = mu + 1
    total = 0.0
    for nu in range(4):
        if nu == mu:
            continue
        for n in (nu + 1, -(nu + 1)):
            for c, path in ((c0, (n, -f, -n)), (c1, (f, n, -f, -f, -n)), (c1, (n, -f, -f, -n, f)),
                            (c1, (n, n, -f, -n, -n))):
                if c:
                    total = total + c * _line_from(u, mu, path)
    return total


def _line_from(u, mu, path):
    """_line starting at x + mu, seen from x."""
    return _at(_line(u, path), (mu, 1))


def _exp(q):
    """Exponential of a field of 3x3 matrices: scaled power series, squared back."""
    q = q / 8.0
    eye = torch.eye(3, dtype=q.dtype, device=q.device).reshape((3, 3) + (1,) * (q.dim() - 2))
    out = term = eye.expand(q.shape)
    for n in range(1, 17):
        term = _mul(term, q) / n
        out = out + term
    for _ in range(3):
        out = _mul(out, out)
    return out


def _traceless_antihermitian(w):
    a = 0.5 * (w - _dag(w))
    tr = (a[0, 0] + a[1, 1] + a[2, 2]) / 3
    eye = torch.eye(3, dtype=a.dtype, device=a.device).reshape((3, 3) + (1,) * (a.dim() - 2))
    return a - tr * eye


def _smear(u, mu):
    """exp(iQ) U for the links of one direction: iQ is the traceless anti-Hermitian part of
    C U^dag, C the weighted sum of the 3-link paths from x to x + mu."""
    f = mu + 1
    c = 0.0
    for nu in range(4):
        if nu != mu:
            for n in (nu + 1, -(nu + 1)):
                c = c + RHO * _line(u, (n, f, -n))
    return _mul(_exp(_traceless_antihermitian(_mul(c, _dag(u[mu])))), u[mu])


def _packed(links, fmt):
    """Links in the order of the format's numbers, as 64-bit reals."""
    if fmt == "c128_18":
        return torch.view_as_real(links.contiguous()).reshape(-1)
    rows = links[:, :2]
    if fmt == "c64_12":          # pairs of entries per 16-byte chunk
        rows = rows.reshape(8, 3, 2, -1).transpose(2, 3)
    return torch.view_as_real(rows.contiguous()).reshape(-1)


def _exact_md(case, seed):
    dims, fmt = _dims(case), case["fmt"]
    lat = _Lattice(dims)
    u = _full(lat, _stored(_links(dims, seed), fmt))
    mom = _momenta(dims, seed)
    if fmt == "c64_12":
        mom = torch.view_as_complex(torch.view_as_real(mom).float().double())
    c1 = -1.0 / 12.0
    force = torch.stack([_traceless_antihermitian(_mul(u[mu], _staple(u, mu, 1 - 8 * c1, c1)))
                         for mu in range(4)])
    # F = -(beta/3) [i U Sigma]_TH, and [iM]_TH = i times the traceless anti-Hermitian part of M
    mom = mom + EPS * (BETA / 3.0) * _slots(lat, 1j * force)
    step = torch.stack([_exp(1j * EPS * m) for m in _full(lat, mom)])
    new = torch.stack([_mul(step[mu], u[mu]) for mu in range(4)])
    return [_packed(_slots(lat, new), fmt), mom]


def _exact_force(case, seed):
    dims = _dims(case)
    lat = _Lattice(dims)
    thin = _full(lat, _stored(_links(dims, seed), case["fmt"]))
    smeared = _slots(lat, torch.stack([_smear(thin, mu) for mu in range(4)]))
    x = _solutions(case, dims, seed)
    y = _Operator(dims, smeared).hop(1, x)
    ph = lat.phases()
    g = torch.zeros_like(smeared)
    for k, a in enumerate(_weights(case)):
        for mu in range(4):
            for par, mine, other, sign in ((0, x[k], y[k], 1.0), (1, y[k], x[k], -1.0)):
                s = 2 * mu + par
                ahead = other[:, lat.near(par, mu, 1)]
                g[s] += sign * a * ph[s] * ahead[:, None] * mine.conj()[None]
    # dS = Re Tr(dU' G) carried to the thin links by automatic differentiation, one
    # direction of the smeared links at a time; grad = (dS/dU)^dag
    gf = _full(lat, g)
    sigma = torch.zeros_like(gf)
    for mu in range(4):
        u = thin.clone().requires_grad_(True)
        s = (_smear(u, mu) * gf[mu].transpose(0, 1)).sum().real
        (grad,) = torch.autograd.grad(s, u)
        sigma += grad.transpose(1, 2).conj()
        del u, s, grad
    return [smeared, y, g, _slots(lat, sigma)]


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        out = []
        for i, (dims, nrhs, mass) in enumerate(_batch_plan(case)):
            op = _Operator(dims, _stored(_links(dims, seed, 8 + i), case["hi"]))
            b = _normal(_gen(seed, 36 + i), nrhs, 3, _half(dims))
            x = _solve(op, mass * mass, b)
            out.append(None if x is None else x[0])
        return out
    dims = _dims(case)
    if kind == "md":
        return _exact_md(case, seed)
    if kind == "force":
        return _exact_force(case, seed)
    if kind == "staples":
        lat = _Lattice(dims)
        u = _full(lat, _stored(_links(dims, seed), case["fmt"]))
        c1 = -1.0 / 12.0
        return _slots(lat, torch.stack([_staple(u, mu, 1 - 8 * c1, c1) for mu in range(4)]))
    links = _links(dims, seed)
    if kind == "operator":
        ph = _phases(dims, seed) if case["phases"] else None
        v = _normal(_gen(seed, 1), case["nrhs"], 3, _half(dims))
        if _field_dtype(case["fmt"]) == torch.complex64:
            v = torch.view_as_complex(torch.view_as_real(v).float().double())
            ph = None if ph is None else ph.float().double()
        op = _Operator(dims, _stored(links, case["fmt"]), ph)
        if case["op"] == "normal":
            return op.normal(0.05 ** 2, v)
        return op.hop(0 if case["op"] == "eo" else 1, v)
    # solves: about 31 / (lightest mass) iterations of some 5 ns per site and right-hand side
    light = case["mass"] if kind == "cg" else math.sqrt(case["mass"] ** 2 + _shifts(case)[0])
    if 40.0 / light * case["nrhs"] * (6e-4 + 3e-9 * _half(dims)) > 15.0:
        return None
    op = _Operator(dims, _stored(links, case["hi"]))
    b = _normal(_gen(seed, 1), case["nrhs"], 3, _half(dims))
    diag = case["mass"] ** 2
    if kind == "cg":
        x = _solve(op, diag, b)
        return None if x is None else x[0]
    x = _solve(op, diag, b, _shifts(case))
    if x is None or case["op"] == "multishift":
        return x
    return 0.3 * b + sum(a * xk for a, xk in zip(_weights(case), x))
