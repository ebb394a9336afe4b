"""The work that programs have this solver do, as cases that can be timed and checked.

A case is a dict of plain values:

  do        "solve"    one solve on a built hierarchy, from x = 0
            "request"  hierarchy setup and one solve, then the hierarchy is released: a served
                       request with a new geometry
            "resetup"  numeric re-setup for a slightly longer pipe on the same lattice and a
                       solve warm-started from the previous one: a step of an elongating bunch
            "step"     a particle-in-cell step: deposition, warm-started solve, field gather
            "batch"    several solves on different geometries advanced together
  shape     "cylinder" (radius 1), "ellipse" (1.0 x 0.6), "boxbore" (0.8 x 0.8 cavity of a third
            of the length, bore radius 0.5)
  nx ny nz  lattice nodes per axis (a batch: of its largest geometry); length of the pipe
  variant   wall rule "const", "lin" or "quad"; precision "fp64" or "mixed"
  open      open (Robin) pipe ends; particles: of the bunch that makes the charge density

``exact`` solves the same discrete problems in plain fp64 torch, from its own geometry and
stencils, by Jacobi-preconditioned BiCGStab to the rounding level.
"""
import math

import torch

import paper_0907_4863_amd as sa
import workloads as W

VARIANTS = {"const": sa.VARIANT_CONST, "lin": sa.VARIANT_LIN, "quad": sa.VARIANT_QUAD}
PRECISIONS = {"fp64": sa.FP64, "mixed": sa.MIXED}
TOL = 1e-8             # relative residual of the scaled system, the solver's default
BATCH = 6              # geometries of a batch
GROWTH = 1.01          # length of the pipe after a re-setup over the one before
STEP_Z = 0.02          # bunch motion per particle-in-cell step
EXACT_NODES = 40_000_000   # larger boxes get no exact solution (time)


def _case(name, do, shape, nx, ny, nz, length, variant, precision, particles, open_ends=False):
    c = {"do": do, "shape": shape, "nx": nx, "ny": ny, "nz": nz, "length": length,
         "variant": variant, "precision": precision, "particles": particles, "open": open_ends}
    return {"name": name, **c} if name else c


def listed():
    return [
        # the smallest solve of the tests and benchmark (33^3 cylinder): a few launches per step
        _case("solve_cyl33_lin_fp64", "solve", "cylinder", 33, 33, 33, 2.0, "lin", "fp64", 20_000),
        # an ordinary beam pipe, nonsymmetric wall rule, all in fp64
        _case("solve_ell128_quad_fp64", "solve", "ellipse", 128, 128, 256, 4.0, "quad", "fp64",
              1_000_000),
        # the benchmark's headline pipe, in both precisions
        _case("solve_ell256_quad_mixed", "solve", "ellipse", 256, 256, 768, 4.0, "quad", "mixed",
              1_000_000),
        _case("solve_ell256_quad_fp64", "solve", "ellipse", 256, 256, 768, 4.0, "quad", "fp64",
              1_000_000),
        # a served cavity of odd size whose hierarchy is resident
        _case("solve_box97_lin_mixed", "solve", "boxbore", 97, 97, 291, 6.0, "lin", "mixed",
              100_000),
        # a large tube with open ends, the constant wall rule
        _case("solve_tube512_const_mixed", "solve", "cylinder", 512, 512, 512, 2.0, "const",
              "mixed", 1_000_000, True),
        # served requests with a new geometry: a small one, and one near the top of the range
        _case("request_cyl64_lin_mixed", "request", "cylinder", 64, 64, 128, 4.0, "lin", "mixed",
              100_000),
        _case("request_ell145_lin_mixed", "request", "ellipse", 145, 145, 435, 6.0, "lin", "mixed",
              100_000),
        # one step of an elongating bunch on the kept aggregation hierarchy
        _case("resetup_ell128_quad_mixed", "resetup", "ellipse", 128, 128, 256, 4.0, "quad",
              "mixed", 1_000_000),
        # particle-in-cell steps: a small open pipe, and a long one with two million particles
        _case("step_cyl49_lin_fp64", "step", "cylinder", 49, 49, 97, 4.0, "lin", "fp64", 100_000,
              True),
        _case("step_cyl192_lin_mixed", "step", "cylinder", 192, 192, 1024, 8.0, "lin", "mixed",
              2_000_000),
        # resident hierarchies of served sizes, their solves advanced together
        _case("batch_box96_lin_mixed", "batch", "boxbore", 96, 96, 192, 4.0, "lin", "mixed",
              100_000),
    ]


def draw(rng):
    """Another case: edges 32..288 over their logarithm, length ratios 1..4 as the served pipes
    have, boxes of at most 40 million nodes."""
    do = rng.choice(["solve", "solve", "solve", "request", "request", "resetup", "step", "step",
                     "batch"])
    hi = {"solve": 288, "request": 224, "resetup": 224, "step": 224, "batch": 112}[do]
    while True:
        e = int(round(math.exp(rng.uniform(math.log(32), math.log(hi)))))
        ratio = rng.choice([1, 2, 3, 4])
        if e * e * e * ratio <= 40_000_000:
            break
    shape = rng.choice(["cylinder", "ellipse", "boxbore"])
    variant = rng.choice(["lin", "lin", "quad", "quad", "const"])
    if do in ("resetup", "batch"):
        # a re-setup keeps the unknowns: pipes that do not vary along z; the batch mixes shapes
        shape = "boxbore" if do == "batch" else rng.choice(["cylinder", "ellipse"])
    precision = rng.choice(["mixed", "mixed", "fp64"])
    particles = int(round(math.exp(rng.uniform(math.log(2e4), math.log(2e6)))))
    return _case("", do, shape, e, e, e * ratio + rng.choice([0, 0, 1]), 2.0 * ratio, variant,
                 precision, particles, do != "batch" and shape != "boxbore" and rng.random() < 0.3)


# ------------------------------------------------------------------ inputs


def _shape(kind, length):
    if kind == "cylinder":
        return W.Shape.cylinder(1.0, length)
    if kind == "ellipse":
        return W.Shape.ellipse(1.0, 0.6, length)
    return W.Shape.boxbore(0.8, length, bore_r=0.5)


def _half(case):
    a, b = {"cylinder": (1.0, 1.0), "ellipse": (1.0, 0.6), "boxbore": (0.8, 0.8)}[case["shape"]]
    return a, b, 0.5 * case["length"]


def _dims(case):
    return case["nx"], case["ny"], case["nz"] + 2 * int(case["open"])


def _bunch(case, seed):
    """Particle positions (n, 3) of a Gaussian bunch near the axis, a little different in place
    and size for each seed."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    a, b, c = _half(case)
    half = torch.tensor([a, b, c], dtype=torch.float64, device="cuda")
    u = torch.rand(6, generator=g, dtype=torch.float64, device="cuda")
    sigma = torch.tensor([0.1, 0.1, 0.15], dtype=torch.float64, device="cuda") * (0.8 + 0.4 * u[:3])
    p = torch.randn(case["particles"], 3, generator=g, dtype=torch.float64, device="cuda")
    return (p * sigma + 0.2 * (u[3:] - 0.5)) * half


def _cells(case, pos, length):
    """Cell (i, j, k) and fractional offset of each particle, and whether it lies in the lattice."""
    a, b, _ = _half(case)
    n = torch.tensor([case["nx"], case["ny"], case["nz"]], device="cuda")
    ext = torch.tensor([2 * a, 2 * b, length], dtype=torch.float64, device="cuda")
    u = (pos + 0.5 * ext) / (ext / (n - 1))
    cell = torch.floor(u).long()
    return cell, u - cell, ((cell >= 0) & (cell <= n - 2)).all(dim=1)


def _corners(case, cell, frac):
    """(box node, trilinear weight) of each of the 8 corners of the particles' cells."""
    nx, ny, _ = _dims(case)
    oz = int(case["open"])
    for k in range(8):
        d = torch.tensor([k & 1, k >> 1 & 1, k >> 2], device="cuda")
        w = torch.where(d.bool(), frac, 1.0 - frac).prod(dim=1)
        c = cell + d
        yield c[:, 0] + nx * (c[:, 1] + ny * (c[:, 2] + oz)), w


def _density(case, pos, length, integer=True):
    """Cloud-in-cell charge density of unit total charge on the box. With ``integer`` the
    weights are summed as multiples of 2^-40, so that the sums do not depend on their order."""
    nx, ny, nz = _dims(case)
    a, b, _ = _half(case)
    cell, frac, ok = _cells(case, pos, length)
    cell, frac = cell[ok], frac[ok]
    rho = torch.zeros(nx * ny * nz, dtype=torch.int64 if integer else torch.float64, device="cuda")
    for node, w in _corners(case, cell, frac):
        rho.index_add_(0, node, torch.round(w * 2.0 ** 40).long() if integer else w)
    vol = 2 * a / (nx - 1) * (2 * b / (ny - 1)) * (length / (case["nz"] - 1))
    rho = rho.double() * 2.0 ** -40 if integer else rho
    return rho / (case["particles"] * vol)


def _domain(case, length=None):
    s = _shape(case["shape"], case["length"] if length is None else length)
    return sa.domain_for(s, case["nx"], case["ny"], case["nz"], case["open"])


def _options(case):
    return sa.default_options(precision=PRECISIONS[case["precision"]])


def _members(case):
    """The geometries of a batch: the shapes of the served stream at falling sizes."""
    out = []
    for k in range(BATCH):
        e = max(24, int(case["nx"] * (1.0 - 0.11 * k)))
        r = case["nz"] / case["nx"]
        out.append(dict(case, shape=("boxbore", "cylinder", "ellipse")[k % 3], nx=e, ny=e,
                        nz=int(e * r)))
    return out


def prepare(case, seed):
    do, var = case["do"], VARIANTS[case["variant"]]
    if do == "batch":
        members = []
        for k, m in enumerate(_members(case)):
            H = sa.setup(_domain(m), var, _options(m))
            b = _density(m, _bunch(m, seed * 16 + k), m["length"])
            members.append((H, b, torch.zeros_like(b), torch.cuda.Stream()))
        torch.cuda.synchronize()
        return {"do": do, "members": members}
    dom = _domain(case)
    st = {"do": do, "dom": dom, "var": var, "opt": _options(case)}
    if do == "step":
        pos = _bunch(case, seed)
        st["H"] = sa.setup(dom, var, st["opt"])
        a, b, c = _half(case)
        st["pic"] = sa.pic_create(dom, (-a, -b, -c), case["particles"])
        st["pos"], st["q"] = pos, 1.0 / case["particles"]
        st["rho"] = torch.zeros(H_nodes(case), dtype=torch.float64, device="cuda")
        st["E"] = torch.zeros_like(pos)
        before = pos - torch.tensor([0.0, 0.0, STEP_Z], dtype=torch.float64, device="cuda")
        first = _density(case, before, case["length"])
    else:
        st["b"] = first = _density(case, _bunch(case, seed), case["length"])
    st["x"] = torch.zeros_like(first)
    if do in ("step", "resetup"):  # the solution of the step before
        if do == "resetup":
            st["H"] = sa.setup(dom, var, st["opt"])
            st["next"] = _domain(case, GROWTH * case["length"])
        st["x0"] = torch.zeros_like(first)
        sa.solve(st["H"], first, st["x0"], tol=TOL)
    elif do == "solve":
        st["H"] = sa.setup(dom, var, st["opt"])
    return st


def H_nodes(case):
    nx, ny, nz = _dims(case)
    return nx * ny * nz


def run(st):
    do = st["do"]
    if do == "batch":
        live = []
        for H, b, x, stream in st["members"]:
            live.append(sa.state_create(H, b, tol=TOL, stream=stream.cuda_stream))
        while sa.batch_step(live) < len(live):
            pass
        for S, (H, b, x, stream) in zip(live, st["members"]):
            sa.state_finish(S, x)
            sa.state_destroy(S)
        return [m[2] for m in st["members"]]
    if do == "request":
        H = sa.setup(st["dom"], st["var"], st["opt"])
        sa.solve(H, st["b"], st["x"], tol=TOL)
        sa.destroy(H)
    elif do == "resetup":
        sa.refresh(st["H"], st["next"])
        sa.solve(st["H"], st["b"], st["x"], x0=st["x0"], tol=TOL)
    elif do == "step":
        sa.pic_deposit(st["pic"], st["pos"], st["q"], st["rho"])
        sa.solve(st["H"], st["rho"], st["x"], x0=st["x0"], tol=TOL)
        sa.pic_gather(st["pic"], st["x"], st["pos"], st["E"])
        return {"rho": st["rho"], "x": st["x"], "E": st["E"]}
    else:
        sa.solve(st["H"], st["b"], st["x"], tol=TOL)
    return {"x": st["x"]}


# ------------------------------------------------------------------ what a pass cannot do without


def work(case):
    """Of a solve: conjugate-gradient steps with one multigrid V-cycle each, whose vectors do not
    fit any cache between two passes over the lattice. A step cannot do with fewer passes than a
    down-stroke (r in, x out), an up-stroke (x and r in, z out), the direction (z and p in, p
    out), the residual (p and r in, r out, and its fp32 copy) and the solution's share of a ring
    of directions: 60 bytes an unknown in mixed precision and 96 in fp64. A setup adds 15
    Lanczos steps of 24 bytes and 28 bytes of domain and scaling, particles 24 bytes of position
    read by each of deposition and gather and 24 of field written."""
    cases = _members(case) if case["do"] == "batch" else [case]
    total = flops = 0.0
    for c in cases:
        n = _fill(c) * c["nx"] * c["ny"] * c["nz"]
        its = {"resetup": 12, "step": 12}.get(case["do"], 12 if n < 1e6 else 18)
        per = 60.0 if c["precision"] == "mixed" else 96.0
        total += n * (its * per + 40.0)
        flops += n * its * 110.0
        if case["do"] in ("request", "resetup"):
            total += n * (15 * 24.0 + 28.0)
            flops += n * 15 * 20.0
        if case["do"] == "step":
            total += case["particles"] * 72.0 + 16.0 * H_nodes(c)
            flops += case["particles"] * 200.0
    return {"bytes": total, "flops": flops}


def _fill(case):
    """Share of the lattice that lies in the pipe."""
    if case["shape"] == "boxbore":
        return 1.0 / 3.0 + 2.0 / 3.0 * math.pi * 0.25 / 2.56
    return math.pi / 4.0


# ------------------------------------------------------------------ the same in plain torch


def _axis(half, n):
    return half * (2.0 * torch.arange(n, dtype=torch.float64, device="cuda") - (n - 1)) / (n - 1)


def _geometry(case, length):
    """Unknowns of the box (nz, ny, nx), and a function giving the distance from every node to the
    wall along +axis or -axis (in units of length; the end of the grid line's interval)."""
    a, b, _ = _half(case)
    nx, ny, nzl = case["nx"], case["ny"], case["nz"]
    X = _axis(a, nx).view(1, 1, nx)
    Y = _axis(b, ny).view(1, ny, 1)
    Z = _axis(0.5 * length, nzl).view(nzl, 1, 1)
    keep = 1.0 - 1e-12
    if case["shape"] == "boxbore":
        cav = length / 6.0
        bore = X * X + Y * Y < 0.25 * keep
        in_cav = Z.abs() < cav * keep
        mask = ((X.abs() < a * keep) & (Y.abs() < b * keep) & in_cav) | bore
        chord = lambda t: torch.where(in_cav, torch.full_like(t, a),  # noqa: E731
                                      torch.sqrt(torch.clamp(0.25 - t * t, min=0.0)))
        ends = [chord(Y), chord(X), torch.where(bore, torch.full_like(X * Y, 0.5 * length),
                                                torch.full_like(X * Y, cav))]
    else:
        inside = X * X + Y * Y < keep if case["shape"] == "cylinder" else (X / a) ** 2 + (Y / b) ** 2 < keep
        mask = inside.expand(nzl, ny, nx)
        ends = [a * torch.sqrt(torch.clamp(1.0 - (Y / b) ** 2, min=0.0)),
                b * torch.sqrt(torch.clamp(1.0 - (X / a) ** 2, min=0.0)),
                torch.full_like(X * Y, 0.5 * length)]
    m = torch.zeros(nzl + 2, ny, nx, dtype=torch.bool, device="cuda")
    m[1:-1, 1:-1, 1:-1] = mask[:, 1:-1, 1:-1]
    if not case["open"]:
        m = m[1:-1].clone()
        m[0] = m[-1] = False
    return m, ends, (X, Y, Z)


def _shift(v, dim, k):
    """v at the next node along dim (k = 1) or the one before (k = -1); 0 beyond the box."""
    out = torch.zeros_like(v)
    n = v.shape[dim]
    if k == 1:
        out.narrow(dim, 0, n - 1).copy_(v.narrow(dim, 1, n - 1))
    else:
        out.narrow(dim, 1, n - 1).copy_(v.narrow(dim, 0, n - 1))
    return out


def _system(case, length):
    """Diagonal, the 6 neighbour coefficients (-x, +x, -y, ...) and the row factors of the
    7-point system with the case's wall rule."""
    m, ends, pos = _geometry(case, length)
    nz, ny, nx = m.shape
    a, b, _ = _half(case)
    h = (2 * a / (nx - 1), 2 * b / (ny - 1), length / (case["nz"] - 1))
    full = lambda v: torch.full((nz, ny, nx), v, dtype=torch.float64, device="cuda")  # noqa: E731
    diag, off = full(0.0), []
    rows = full(1.0)
    if case["open"]:
        rows[1] = rows[-2] = 0.5
    for ax in range(3):
        dim = 2 - ax
        end = ends[ax]
        lat = torch.zeros((nz, ny, nx), dtype=torch.float64, device="cuda")
        s = []
        for sign in (-1.0, 1.0):  # the wall on either side, in units of the spacing
            d = ((sign * end - pos[ax]).abs() / h[ax]).expand(case["nz"], ny, nx)
            d = torch.where(d > 1.0 - 1e-12, torch.ones_like(d), d)
            lat = full(1.0)
            (lat[1:-1] if case["open"] else lat).copy_(d)
            s.append(lat)
        in_m, in_p = _shift(m, dim, -1), _shift(m, dim, 1)
        sm, sp = s
        sm = torch.where(in_m | ~m, torch.ones_like(sm), sm)
        sp = torch.where(in_p | ~m, torch.ones_like(sp), sp)
        cs, cm, cp = full(2.0), -in_m.double(), -in_p.double()
        if case["variant"] == "lin":
            cs = cs - torch.where(in_m, 0.0, 1.0 - 1.0 / sm) - torch.where(in_p, 0.0, 1.0 - 1.0 / sp)
        elif case["variant"] == "quad":
            one_m, one_p, both = ~in_m & in_p, ~in_p & in_m, ~in_m & ~in_p
            cs = cs - torch.where(one_m, 2.0 * (sm - 1.0) / sm, 0.0) \
                - torch.where(one_p, 2.0 * (sp - 1.0) / sp, 0.0) \
                - torch.where(both, ((sm - 1.0) * (sp + 1.0) + (sm + 1.0) * (sp - 1.0)) / (sm * sp), 0.0)
            cp = cp + torch.where(one_m, (sm - 1.0) / (sm + 1.0), 0.0)
            cm = cm + torch.where(one_p, (sp - 1.0) / (sp + 1.0), 0.0)
        if ax == 2 and case["open"]:  # the open ends: u(x') = u(x'') - (2 h / d) u(x)
            w = 2.0 + 2.0 * h[2] / (0.5 * length)
            cs[1] = cs[-2] = w
            cm[1], cp[1], cm[-2], cp[-2] = 0.0, -2.0, -2.0, 0.0
        ih2 = 1.0 / (h[ax] * h[ax])
        diag += rows * cs * ih2
        off += [torch.where(m & in_m, rows * cm * ih2, 0.0), torch.where(m & in_p, rows * cp * ih2, 0.0)]
    return m, diag, off, rows, h


def _exact_solve(case, b, length):
    """The solution of the discrete problem, by BiCGStab on the unit-diagonal system."""
    m, diag, off, rows, _ = _system(case, length)
    sig = torch.where(m, 1.0 / torch.sqrt(diag), 0.0)
    for k in range(6):
        off[k] *= sig * _shift(sig, 2 - k // 2, 1 if k % 2 else -1)
    rhs = sig * rows * torch.where(m, b.view(m.shape), 0.0)
    del diag, rows

    def apply(v):
        y = v.clone()
        for k in range(6):
            dim, n = 2 - k // 2, v.shape[2 - k // 2]
            lo, hi = (0, 1) if k % 2 else (1, 0)
            y.narrow(dim, lo, n - 1).addcmul_(off[k].narrow(dim, lo, n - 1), v.narrow(dim, hi, n - 1))
        return y

    dot = lambda u, v: torch.dot(u.reshape(-1), v.reshape(-1))  # noqa: E731
    x = torch.zeros_like(rhs)
    goal = 1e-12 * float(rhs.norm())
    for _ in range(4):  # restarted from the true residual
        r = rhs - apply(x)
        if float(r.norm()) <= goal:
            break
        r0, p = r.clone(), r.clone()
        rho = dot(r0, r)
        for it in range(6000):
            v = apply(p)
            alpha = rho / dot(r0, v)
            s = r - alpha * v
            t = apply(s)
            omega = dot(t, s) / dot(t, t)
            x += alpha * p + omega * s
            r = s - omega * t
            new = dot(r0, r)
            if it % 16 == 15 and not float(r.norm()) > 0.3 * goal:
                break
            p = r + (new / rho) * (alpha / omega) * (p - omega * v)
            rho = new
    return (sig * x).reshape(-1)


def _exact_gather(case, phi, pos):
    """E = -grad(phi) at the particles: trilinear interpolation of nodal central differences."""
    m, _, _ = _geometry(case, case["length"])
    a, b, c = _half(case)
    h = (2 * a / (case["nx"] - 1), 2 * b / (case["ny"] - 1), 2 * c / (case["nz"] - 1))
    p = torch.where(m, phi.view(m.shape), 0.0)
    cell, frac, ok = _cells(case, pos, case["length"])
    cell = torch.where(ok[:, None], cell, 0)
    E = torch.zeros_like(pos)
    for ax in range(3):
        q = p
        if ax == 2 and case["open"]:  # beyond the open ends
            r = 2.0 * h[2] / c
            q = p.clone()
            q[0] = torch.where(m[1], p[2] - r * p[1], 0.0)
            q[-1] = torch.where(m[-2], p[-3] - r * p[-2], 0.0)
        g = ((_shift(q, 2 - ax, -1) - _shift(q, 2 - ax, 1)) / (2.0 * h[ax])).reshape(-1)
        for node, w in _corners(case, cell, frac):
            E[:, ax] += torch.where(ok, w * g[node], 0.0)
    return E


def exact(case, seed):
    if H_nodes(case) > EXACT_NODES:
        return None
    if case["do"] == "batch":
        return [_exact_solve(m, _density(m, _bunch(m, seed * 16 + k), m["length"]), m["length"])
                for k, m in enumerate(_members(case))]
    pos = _bunch(case, seed)
    if case["do"] == "step":
        rho = _density(case, pos, case["length"], integer=False)
        x = _exact_solve(case, rho, case["length"])
        return {"rho": rho, "x": x, "E": _exact_gather(case, x, pos)}
    length = case["length"] * (GROWTH if case["do"] == "resetup" else 1.0)
    return {"x": _exact_solve(case, _density(case, pos, case["length"]), length)}
