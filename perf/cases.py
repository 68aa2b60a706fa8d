"""The work that programs have this framework do, as cases to time.

Each case is one pass through the public entry points (Tracker, DepositFn) as
a fluid solver, an optimiser or an output routine calls them, on seeded
synthetic inputs: Taylor-Green-like fields with cell noise, droplets uniform
or in Gaussian plumes, lognormal diameters around 20 um, at rest.

Kinds of pass:
  loop     `steps` times: one step, then the sources taken and cleared, as the
           fluid solver needs them after every step (and, with `ec`, the
           extrapolator-corrector's estimate); with `readout` the particles at
           the end.  The field is another one every 32 steps, as a solver's
           field changes, so droplets keep mixing however long a run is.
  coupled  `steps` steps of the run with the rotating field on its own stream,
           then the sources.
  taped    `steps` taped steps, the sources, and the adjoint of a weighted sum
           of them: the gradients to the field and the diameters.
  deposit  one iteration of a torch optimisation: a fresh tracker, DepositFn
           forward and backward.
  start    a program's start: a fresh tracker, its droplets put in, their
           state and the partitions' bounding boxes read back.
  output   a step, then the particles and the bounding boxes, as a program that
           writes its state does.
  hilbert  positions of new droplets along the Hilbert curve.
"""
import math

import torch

from paper_2603_26691_amd import DepositFn, Tracker
from paper_2603_26691_amd.autograd import Run

DEV = "cuda"
F64 = torch.float64
L = 0.1                    # domain edge along x [m]; the cells are cubes
RHO_F, MU_F, RHO_P, GZ = 1.2, 1.8e-5, 1000.0, -9.81
BATCH = 1 << 24            # droplets drawn (and checked) at a time
FIELD_EVERY, FIELDS = 32, 4

BASE = dict(kind="loop", nx=64, ny=64, nz=64, edge=8, P=100_000, form="fp32_local",
            interp="trilinear", drag="stokes", dt=5e-5, nsub=1, steps=1, noise=0.1, plumes=0,
            share=1.0, tape=0, ec="", readout=False, host=False, parts=1)


def _case(name, **kw):
    return dict(BASE, name=name, **kw)


def listed():
    return [
        # the smallest call: a two-way coupled test flow, where launches and
        # latency count; the estimate that stands in for the late source
        _case("two_way_16", nx=16, ny=16, nz=16, edge=4, P=2000, form="fp64", ec="linear",
              noise=0.0),
        # the plain method in binary64 on a small mesh
        _case("step_32_fp64", nx=32, ny=32, nz=32, P=100_000, form="fp64", dt=1e-4, noise=0.0),
        # ragged mesh and count, the paper's own interpolation and sub-steps,
        # Schiller-Naumann drag, everything in binary32; output every 10 steps
        _case("run_ragged_fp32", nx=48, ny=72, nz=40, P=777_777, form="fp32", interp="ngp",
              drag="schiller_naumann", nsub=2, steps=10, readout=True),
        # the method at scale, uniform droplets
        _case("step_128", nx=128, ny=128, nz=128, P=10_000_000),
        # the same in binary64 with Schiller-Naumann drag
        _case("step_128_fp64_sn", nx=128, ny=128, nz=128, P=10_000_000, form="fp64",
              drag="schiller_naumann"),
        # plumes on a large mesh: strongly uneven chunks
        _case("step_plume_256", nx=256, ny=256, nz=256, P=200_000_000, plumes=4),
        # the largest: the asynchronously coupled run, most droplets in one plume
        _case("coupled_512", kind="coupled", nx=512, ny=512, nz=512, P=400_000_000, plumes=1,
              share=0.6, steps=4),
        # differentiation: forward with checkpoints every 20 steps and adjoint
        _case("adjoint_64", kind="taped", P=1_000_000, steps=40, tape=20, noise=0.0),
        # an optimiser's iteration through torch.autograd, binary64, ragged
        _case("deposit_fn_fp64", kind="deposit", nx=40, ny=48, nz=56, P=100_003, form="fp64",
              drag="schiller_naumann", steps=30, tape=10),
        # start of a program
        _case("start_3e6", kind="start", nx=96, ny=96, nz=96, P=3_000_000, plumes=2, parts=512),
        # output of the full state
        _case("output_1e7", kind="output", nx=128, ny=128, nz=128, P=10_000_000, parts=4096),
        # placement along the Hilbert curve, a segment per 8^3-cell chunk
        _case("hilbert_1e7", kind="hilbert", nx=128, ny=128, nz=128, P=4096 * 2441, parts=4096),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    c = dict(BASE)
    c["kind"] = kind = rng.choice(["loop"] * 4 + ["coupled", "taped", "taped", "deposit", "start",
                                                  "output", "hilbert"])
    c["form"] = rng.choice(["fp32_local", "fp32_local", "fp64"] if kind in ("taped", "deposit")
                           else ["fp32_local", "fp32_local", "fp32_local", "fp64", "fp32"])
    c["edge"] = rng.choice([8, 8, 8, 4])
    c["interp"] = rng.choice(["trilinear", "trilinear", "ngp"])
    c["drag"] = rng.choice(["stokes", "schiller_naumann"])
    c["noise"] = rng.choice([0.0, 0.1])
    c["dt"] = rng.choice([5e-5, 1e-4])
    c["plumes"] = rng.choice([0, 0, 1, 4])
    c["share"] = rng.choice([0.6, 1.0])
    small = kind in ("taped", "deposit")
    edges = [max(2, _log_int(rng, 2, 10 if small else 30)) for _ in range(3)]   # in blocks of 8
    c["nx"], c["ny"], c["nz"] = (8 * e for e in edges)
    cells = c["nx"] * c["ny"] * c["nz"]
    hi = {"taped": 2_000_000, "deposit": 300_000}.get(kind, 60_000_000)
    c["P"] = max(1000, min(hi, int(cells * math.exp(rng.uniform(math.log(0.3), math.log(12))))))
    if kind == "loop":
        c["nsub"] = rng.choice([1, 1, 1, 3])
        c["steps"] = rng.choice([1, 1, 7]) if c["P"] < 5_000_000 else 1
        c["ec"] = rng.choice(["", "", "const", "linear"])
        c["readout"] = c["P"] < 5_000_000 and rng.random() < 0.4
    elif kind == "coupled":
        c["steps"] = rng.choice([2, 5])
    elif small:
        c["steps"], c["tape"] = rng.randint(8, 40), rng.choice([5, 10, 20])
    elif kind in ("start", "output", "hilbert"):
        c["parts"] = _log_int(rng, 1, 4096)
        c["host"] = kind != "output" and c["P"] < 3_000_000 and rng.random() < 0.3
        if kind == "hilbert":
            c["P"] = max(1, c["P"] // c["parts"]) * c["parts"]
    return c


# ---------------------------------------------------------------------------
# inputs, from the seed alone
# ---------------------------------------------------------------------------
def _gen(seed, what):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1_000_003 + what) % (1 << 62))
    return g


def _n(c):
    return c["nx"], c["ny"], c["nz"]


def _extent(c):
    return tuple(L * v / c["nx"] for v in _n(c))


def _tdtype(c):
    return F64 if c["form"] == "fp64" else torch.float32


def _field(c, seed, k):
    """Taylor-Green-like cell-centred field number k, shifted by phases of its
    own, [3, nz, ny, nx] in the form's field precision."""
    g = _gen(seed, 100 + k)
    ph = 2 * math.pi * torch.rand(3, dtype=F64, device=DEV, generator=g)
    a = [2 * math.pi * (torch.arange(n, dtype=F64, device=DEV) + 0.5) / n + p
         for n, p in zip(_n(c), ph)]
    sx, cx = a[0].sin()[None, None, :], a[0].cos()[None, None, :]
    sy, cy = a[1].sin()[None, :, None], a[1].cos()[None, :, None]
    cz = a[2].cos()[:, None, None]
    U = torch.stack([cz * cy * sx, -cz * sy * cx, torch.zeros_like(cz * cy * sx)])
    if c["noise"] > 0:
        U += c["noise"] * torch.randn(U.shape, dtype=torch.float32, device=DEV, generator=g)
    return U.to(_tdtype(c)).contiguous()


def _weights(c, seed):
    return torch.randn((3, c["nz"], c["ny"], c["nx"]), dtype=F64, device=DEV,
                       generator=_gen(seed, 7))


def _batches(c, seed):
    """(x, up, d) of BATCH droplets at a time, binary64 on the device."""
    ext = torch.tensor(_extent(c), dtype=F64, device=DEV)
    centres = torch.rand((max(c["plumes"], 1), 3), dtype=F64, device=DEV,
                         generator=_gen(seed, 1)) * ext
    for b in range(-(-c["P"] // BATCH)):
        k = min(c["P"] - b * BATCH, BATCH)
        g = _gen(seed, 1000 + b)
        x = torch.rand((k, 3), dtype=F64, device=DEV, generator=g) * ext
        if c["plumes"]:
            inside = torch.rand(k, device=DEV, generator=g) < c["share"]
            which = torch.randint(0, c["plumes"], (k,), device=DEV, generator=g)
            off = torch.randn((k, 3), dtype=F64, device=DEV, generator=g) * (0.05 * ext)
            x = torch.where(inside[:, None], torch.remainder(centres[which] + off, ext), x)
            x = torch.where(x >= ext, torch.zeros_like(x), x)
        d = torch.exp(math.log(20e-6) +
                      0.4 * torch.randn(k, dtype=F64, device=DEV, generator=g))
        yield x, torch.zeros_like(x), d


def _whole(c, seed):
    x, up, d = zip(*_batches(c, seed))
    return torch.cat(x), torch.cat(up), torch.cat(d)


def _uniforms(c, seed):
    return torch.rand((c["P"], 3), dtype=F64, device=DEV, generator=_gen(seed, 5))


def _order(c):
    return max(1, round(math.log2(c["nx"])))


def _angles(c, first):
    """(cos, sin) of the field's rotation, one degree a step, from step `first`."""
    th = [math.radians(first + k) for k in range(c["steps"])]
    return [v for t in th for v in (math.cos(t), math.sin(t))]


def _tracker(c):
    return Tracker(_n(c), _extent(c), c["P"], form=c["form"], interp=c["interp"],
                   chunk_edge=c["edge"], rho_f=RHO_F, mu_f=MU_F, g=(0.0, 0.0, GZ), rho_p=RHO_P,
                   drag=c["drag"])


def _per_part(c):
    return -(-c["P"] // c["parts"])


def prepare(case, seed):
    c = case
    s = {"case": c, "pass": 0}
    kind = c["kind"]
    if kind == "hilbert":
        s["tracker"] = Tracker(_n(c), _extent(c), 1, chunk_edge=c["edge"])
        s["u"] = _uniforms(c, seed)
        if c["host"]:
            s["u"] = s["u"].cpu().numpy()
        return s
    if kind in ("deposit", "start"):
        s["x"], s["up"], s["d"] = _whole(c, seed)
        if c["host"]:
            s["x"], s["up"], s["d"] = (v.cpu().numpy() for v in (s["x"], s["up"], s["d"]))
        if kind == "deposit":
            s["U"] = _field(c, seed, 0).to(F64).requires_grad_(True)
            s["d"].requires_grad_(True)
            s["w"] = _weights(c, seed)
        return s
    t = s["tracker"] = _tracker(c)
    for x, up, d in _batches(c, seed):
        t.inject(x, up, d)
    s["fields"] = [_field(c, seed, k) for k in range(FIELDS if kind in ("loop", "output") else 1)]
    if kind == "taped":
        s["w"] = _weights(c, seed)
    return s


def run(state):
    c = state["case"]
    kind, dt = c["kind"], c["dt"]
    k = state["pass"]
    state["pass"] = k + 1
    if kind == "loop":
        t, S, out = state["tracker"], [], {}
        for j in range(c["steps"]):
            U = state["fields"][(k * c["steps"] + j) // FIELD_EVERY % FIELDS]
            t.step(U, dt, nsub=c["nsub"])
            S.append(t.sources(reset=True))
            if c["ec"]:
                S[-1] = t.ec_estimate(c["ec"], S[-1])
        out["S"] = S
        if c["readout"]:
            out.update(t.particles())
        return out
    if kind == "coupled":
        t = state["tracker"]
        t.run_coupled(state["fields"][0], _angles(c, k * c["steps"]), dt, timed=False)
        return t.sources(reset=True)
    if kind == "taped":
        t, U = state["tracker"], state["fields"][0]
        for _ in range(c["steps"]):
            t.step(U, dt, nsub=c["nsub"], tape=c["tape"])
        S = t.sources(reset=True)
        dU, dd = t.backward(state["w"])
        return {"S": S, "dU": dU, "dd": dd}
    if kind == "deposit":
        t = _tracker(c)
        S = DepositFn.apply(state["U"], state["d"],
                            Run(t, state["x"], state["up"], dt, c["steps"], tape_every=c["tape"]))
        loss = (state["w"] * S).sum()
        dU, dd = torch.autograd.grad(loss, (state["U"], state["d"]))
        t.close()
        return {"S": S.detach(), "dU": dU, "dd": dd}
    if kind == "start":
        t = _tracker(c)
        t.inject(state["x"], state["up"], state["d"])
        out = t.particles()
        out["boxes"] = t.bounding_boxes(0, _per_part(c), c["parts"])
        t.close()
        return out
    if kind == "output":
        t = state["tracker"]
        t.step(state["fields"][k // FIELD_EVERY % FIELDS], dt)
        out = t.particles()
        out["boxes"] = t.bounding_boxes(0, _per_part(c), c["parts"])
        return out
    return state["tracker"].hilbert_positions(_order(c), c["parts"], 0, c["parts"],
                                              c["P"] // c["parts"], state["u"])


def work(case):
    """Bytes that a pass cannot do without: per step each droplet's position,
    velocity and diameter read, position and velocity written, the field read
    and the sources written; per reversed step the state read and the adjoint
    state (seven values) read and written; inputs and outputs once."""
    c = case
    P, cells, kind = c["P"], c["nx"] * c["ny"] * c["nz"], c["kind"]
    ts = 8 if c["form"] == "fp64" else 4
    step = P * 13 * ts + 3 * cells * ts
    gather = 90 if c["interp"] == "trilinear" else 20
    flops = P * (gather + 40 + (20 if c["drag"] != "stokes" else 0))
    sources, state_in, state_out = 24 * cells, 56 * P, 76 * P
    if kind == "hilbert":
        return {"bytes": 48 * P, "flops": 6 * P}
    if kind == "start":
        return {"bytes": state_in + state_out + 48 * c["parts"], "flops": 20 * P}
    if kind == "output":
        return {"bytes": step + state_out + 48 * c["parts"], "flops": flops}
    n = c["steps"] * c["nsub"]
    if kind in ("taped", "deposit"):
        back = P * (7 + 14) * ts + 3 * cells * ts
        total = n * (step + back) + 3 * sources + 8 * P
        return {"bytes": total + (state_in if kind == "deposit" else 0), "flops": 3.5 * n * flops}
    once = state_out if c["readout"] else 0
    per = 3 if c["ec"] else 1
    return {"bytes": n * step + (1 if kind == "coupled" else c["steps"]) * per * sources + once,
            "flops": n * flops}


# ---------------------------------------------------------------------------
# the same results in plain torch, 64 bits
# ---------------------------------------------------------------------------
def _advance(c, U, x, up, d, dt):
    """One step of some droplets: the new (x, up), and the cells and values of
    their sources.  U: [cells, 3]."""
    n = torch.tensor(_n(c), device=DEV)
    ext = torch.tensor(_extent(c), dtype=F64, device=DEV)
    h = ext / n
    flat = lambda i: (i[:, 2] * n[1] + i[:, 1]) * n[0] + i[:, 0]  # noqa: E731
    g = x / h
    cell = flat(torch.remainder(g.detach().floor().long(), n))
    if c["interp"] == "trilinear":
        i0 = (g.detach() - 0.5).floor()
        f = g - 0.5 - i0
        i0 = i0.long()
        uf = 0.0
        for k in range(8):
            b = [(k >> a) & 1 for a in range(3)]
            w = math.prod(f[:, a] if b[a] else 1.0 - f[:, a] for a in range(3))
            idx = flat(torch.remainder(i0 + torch.tensor(b, device=DEV), n))
            uf = uf + w[:, None] * U.index_select(0, idx)
    else:
        uf = U.index_select(0, cell)
    grav = torch.tensor((0.0, 0.0, GZ), dtype=F64, device=DEV)
    tau = RHO_P * d * d / (18.0 * MU_F)
    slip = uf - up
    if c["drag"] != "stokes":
        re2 = (RHO_F / MU_F * d) ** 2 * (slip * slip).sum(1)
        tau = tau / (1.0 + 0.15 * re2 ** 0.3435)
    new = up + (dt / (tau + dt))[:, None] * (slip + tau[:, None] * grav)
    m = RHO_P * math.pi / 6.0 * d ** 3
    src = -(m[:, None] * (new - up - grav * dt)) / h.prod()
    x = x + dt * new
    x = x - (x.detach() / ext).floor() * ext
    return x, new, cell, src


def _sources(c, S):
    return S.t().reshape(3, c["nz"], c["ny"], c["nx"])


def _rows(U):
    return U.to(F64).reshape(3, -1).t().contiguous()


def _boxes(c, x):
    per, parts = _per_part(c), c["parts"]
    part = torch.arange(c["P"], device=DEV) // per
    at = part[:, None].expand(-1, 3)
    lo = torch.full((parts, 3), math.inf, dtype=F64, device=DEV).scatter_reduce(0, at, x, "amin")
    hi = torch.full((parts, 3), -math.inf, dtype=F64, device=DEV).scatter_reduce(0, at, x, "amax")
    return torch.cat([lo, hi], 1)


def _particles(x, up, d):
    return {"x": x, "up": up, "d": d, "id": None, "cell": None}


def _exact_steps(c, fields, x, up, d):
    """Steps over the fields (in sub-steps), droplets BATCH at a time: the
    state after them (in place) and each step's sources."""
    out = []
    for U in fields:
        U = _rows(U)
        S = torch.zeros_like(U)
        for _ in range(c["nsub"]):
            for b in range(0, c["P"], BATCH):
                q = slice(b, b + BATCH)
                xn, un, cell, src = _advance(c, U, x[q], up[q], d[q], c["dt"] / c["nsub"])
                x[q], up[q] = xn, un
                S.index_add_(0, cell, src)
        out.append(S)
    return [_sources(c, S) for S in out]


def exact(case, seed):
    c = case
    kind = c["kind"]
    if kind == "hilbert":
        return None     # whole-number curve positions; the tests pin them bit for bit
    x, up, d = _whole(c, seed)
    if kind == "start":
        return dict(_particles(x, up, d), boxes=_boxes(c, x))
    if kind in ("taped", "deposit"):
        U = _field(c, seed, 0).to(F64).requires_grad_(True)
        d.requires_grad_(True)
        rows = U.reshape(3, -1).t()
        S = torch.zeros_like(rows)
        for _ in range(c["steps"] * c["nsub"]):
            x, up, cell, src = _advance(c, rows, x, up, d, c["dt"] / c["nsub"])
            S = S.index_add(0, cell, src)
        S = _sources(c, S)
        dU, dd = torch.autograd.grad((S * _weights(c, seed)).sum(), (U, d))
        return {"S": S.detach(), "dU": dU, "dd": dd}
    if kind == "coupled":
        U0 = _field(c, seed, 0).to(F64)
        cs = _angles(c, 0)
        rot = (torch.stack([a * U0[0] - b * U0[1], b * U0[0] + a * U0[1], U0[2]])
               for a, b in zip(cs[0::2], cs[1::2]))
        return sum(_exact_steps(c, rot, x, up, d))
    if kind == "output":
        _exact_steps(c, [_field(c, seed, 0)], x, up, d)
        return dict(_particles(x, up, d), boxes=_boxes(c, x))
    S = _exact_steps(c, [_field(c, seed, j // FIELD_EVERY % FIELDS) for j in range(c["steps"])],
                     x, up, d)
    if c["ec"]:
        prev, last, got = torch.zeros_like(S[0]), torch.zeros_like(S[0]), []
        for s in S:
            e = s if c["ec"] == "const" else 2.0 * s - last
            got.append(s - prev + e)
            prev, last = e, s
        S = got
    out = {"S": S}
    if c["readout"]:
        out.update(_particles(x, up, d))
    return out
