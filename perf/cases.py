"""Timed workloads of the thermal lattice Boltzmann library, through its public
Python entry points, and what plain 64-bit arithmetic gives for the same inputs.

A case is one piece of work a user's program has the library do:

  solve    advance one simulation by a number of steps and read its fields (or,
           with F16 storage, its checkpoint): the library's everyday use;
  watch    a few steps, then every diagnostic (conservation totals, fields,
           heat flux);
  begin    set a simulation up from fields that are on the GPU, apply its force,
           take the first step and read the fields;
  restart  checkpoint one simulation and resume it in another;
  batch    advance several grids of different sizes together;
  serve    the continuous-batching server over a queue of requests, set-up,
           stepping and results included.

Grids are rows of x, then y, then z: cell = (z*ny + y)*nx + x.
"""
import math

import numpy as np
import torch

from paper_2302_04741_amd import serve, sim, workloads

DIM = {"D2Q37": 2, "D3Q39": 3}
BYTES = {"f64": 8, "f32": 4, "f16dev": 2}


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def _case(kind, lattice, storage, dims, steps, force="axis", **more):
    nx, ny, nz = (tuple(dims) + (1, 1))[:3]
    return {"kind": kind, "lattice": lattice, "storage": storage, "nx": nx, "ny": ny, "nz": nz,
            "steps": steps, "force": force, **more}


def listed():
    named = [
        # the paper's channel between plates: the smallest production run, a
        # long chain of steps on 450 cells where the latency of a step counts
        ("channel_3x150_f64", _case("solve", "D2Q37", "f64", (3, 150), 100, "channel")),
        # the parity grid, sampled every 20 steps: launches and latency
        ("parity_64_f64", _case("solve", "D2Q37", "f64", (64, 64), 20, "uniform")),
        # one small request of the serving stream, solved alone
        ("shear_256_f32", _case("solve", "D2Q37", "f32", (256, 256), 25)),
        # the thermal shear layer, the usual 2-D production size
        ("shear_1024_f32", _case("solve", "D2Q37", "f32", (1024, 1024), 20)),
        # a ragged 2-D grid in full precision, with every diagnostic
        ("ragged_1537x1021_f64", _case("watch", "D2Q37", "f64", (1537, 1021), 5)),
        # the 3-D Kolmogorov flow, the flagship step, in both reduced storages
        ("kolmogorov_256_f32", _case("solve", "D3Q39", "f32", (256, 256, 256), 10)),
        ("kolmogorov_256_f16", _case("solve", "D3Q39", "f16dev", (256, 256, 256), 10)),
        # an odd 3-D grid in full precision under a force field
        ("field_129x95x110_f64", _case("solve", "D3Q39", "f64", (129, 95, 110), 8, "field")),
        # setting a simulation up and taking its first step
        ("begin_160_f32", _case("begin", "D3Q39", "f32", (160, 160, 160), 1)),
        # checkpoint and restart of a grid whose rows are not whole lines
        ("restart_1017_f32", _case("restart", "D2Q37", "f32", (1017, 1017), 1)),
        # sixteen small independent grids advanced together
        ("batch_16_f32", _case("batch", "D2Q37", "f32", (32, 256), 25, count=16)),
        # the server over a queue of requests, four resident at a time
        ("serve_8_f32", _case("serve", "D2Q37", "f32", (64, 640), 75, "uniform", count=8)),
    ]
    return [{"name": name, **c} for name, c in named]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve", "solve", "solve", "solve", "channel", "watch", "begin", "restart",
                       "batch", "serve"])
    if kind == "channel":
        return _case("solve", "D2Q37", rng.choice(["f64", "f64", "f32"]),
                     (_log_int(rng, 1, 64), rng.randint(60, 300)), rng.randint(20, 100), "channel")
    if kind in ("batch", "serve"):
        lo = _log_int(rng, 16, 64)
        return _case(kind, "D2Q37", rng.choice(["f32", "f32", "f64"]),
                     (lo, _log_int(rng, 96, 400)), rng.randint(10, 50),
                     "axis" if kind == "batch" else "uniform",
                     count=rng.randint(2, 16 if kind == "batch" else 8))
    lattice = rng.choice(["D2Q37", "D3Q39"])
    storage = rng.choice(["f32", "f64", "f16dev"] if kind in ("solve", "restart")
                         else ["f64"] if kind == "watch" else ["f32", "f64"])
    if lattice == "D2Q37":
        dims = (_log_int(rng, 12, 2100), _log_int(rng, 12, 2100))
    else:
        dims = (_log_int(rng, 8, 220), _log_int(rng, 8, 220), _log_int(rng, 8, 220))
    # no more memory traffic than the largest listed case
    most = int(4e10 // (math.prod(dims) * 78 * BYTES[storage]))
    steps = 1 if kind in ("begin", "restart") else max(1, min(rng.randint(1, 12), most))
    return _case(kind, lattice, storage, dims, steps, rng.choice(["axis", "uniform", "field"]))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _problem(case, seed, dims=None, member=0):
    """Fields and force of one simulation from the seed: smooth random fields of
    a few Fourier modes (density within 2%, temperature within 5%, velocities of
    a few hundredths of the reference speed) and a weak body force."""
    lattice = case["lattice"]
    D = DIM[lattice]
    nx, ny, nz = dims or (case["nx"], case["ny"], case["nz"])
    rng = np.random.default_rng([int(seed), int(member)])
    dev = _device()
    kw = {"dtype": torch.float64, "device": dev}
    tx = torch.arange(nx, **kw) * (2 * math.pi / nx)
    ty = torch.arange(ny, **kw) * (2 * math.pi / ny)
    tz = torch.arange(nz, **kw) * (2 * math.pi / nz)

    def smooth(amp):
        out = torch.zeros((nz, ny, nx), **kw)
        for _ in range(3):
            k = rng.integers(0, 3, size=3)
            if not k[:D].any():
                k[rng.integers(0, D)] = 1
            a, ph = rng.uniform(0.3, 1.0) * rng.choice([-1.0, 1.0]), rng.uniform(0, 2 * math.pi)
            arg = k[0] * tx[None, None, :] + k[1] * ty[None, :, None] + ph
            if D == 3:
                arg = arg + k[2] * tz[:, None, None]
            out = out + a * torch.sin(arg)
        return (amp / 3.0) * out

    p = {"lattice": lattice, "storage": case["storage"], "dims": (nx, ny, nz), "mu": 0.0,
         "walls": None, "tau": float(rng.uniform(0.6, 0.9))}
    if case["force"] == "channel":
        # the paper's channel (Sec. 3): U_c = 1.5 and Re = 1800 at any height,
        # started like a channel at rest (uniform along x, as the flow stays)
        hot = float(rng.uniform(1.2, 1.5))
        wl = workloads.channel(0.7, hot, nx=nx, ny=ny)
        p["mu"], p["walls"], g = wl.mu, wl.walls, wl.force[1]
        eta = (torch.arange(ny, **kw) + 0.5) / ny

        def rows(v):
            return v[None, :, None].expand(nz, ny, nx).reshape(-1).contiguous()

        p["theta"] = rows(0.7 + (hot - 0.7) * eta)
        p["rho"] = rows(1.0 + rng.uniform(0.0, 0.02) * torch.cos(2 * math.pi * eta))
        p["u"] = torch.stack([rows(rng.uniform(0.0, 0.1) * eta * (1 - eta)), rows(0.0 * eta)])
        p["force"] = ("uniform", np.asarray(g, dtype=np.float64))
        return p
    p["rho"] = 1.0 + smooth(0.02).reshape(-1)
    p["theta"] = 1.0 + smooth(0.05).reshape(-1)
    p["u"] = torch.stack([smooth(0.05).reshape(-1) for _ in range(D)])
    if case["force"] == "uniform":
        p["force"] = ("uniform", 1e-7 * rng.uniform(-1, 1, size=D))
    elif case["force"] == "axis":
        # Kolmogorov forcing: along x, a sine of the slowest coordinate
        n = (nx, ny, nz)[D - 1]
        prof = np.zeros((D, n))
        prof[0] = 1e-5 * np.sin(2 * math.pi * np.arange(n) / n + rng.uniform(0, 6.28))
        p["force"] = ("axis", D - 1, prof)
    else:
        p["force"] = ("field", torch.stack([smooth(1e-5).reshape(-1) for _ in range(D)]))
    return p


def _sizes(case):
    """Sides of the members of a batch or of the requests of a queue: spread
    evenly over the range, large and small ones mixed."""
    lo, hi, n = case["nx"], case["ny"], case["count"]
    order = sorted(range(n), key=lambda k: (k * 5) % n)
    return [lo + (hi - lo) * k // max(1, n - 1) for k in order]


def _members(case, seed):
    return [_problem(case, seed, (side, side, 1), k)
            for k, side in enumerate(_sizes(case))]


def _request_steps(case, k):
    return case["steps"] + 5 * k  # requests end at different times


def _apply_force(s, p):
    kind = p["force"][0]
    if kind == "uniform":
        s.set_force(p["force"][1])
    elif kind == "axis":
        s.set_force(axis=p["force"][1], profile=p["force"][2])
    else:
        s.set_force(field=p["force"][1])


def _sim(p):
    s = sim.Sim(p["lattice"], p["dims"], p["tau"], p["rho"], p["u"], p["theta"],
                storage=p["storage"], force_field=p["force"][0] == "field",
                walls=p["walls"] is not None)
    if p["mu"] > 0:
        s.set_viscosity(p["mu"])
    _apply_force(s, p)
    if p["walls"] is not None:
        s.set_walls(*p["walls"])
    return s


def prepare(case, seed):
    kind = case["kind"]
    if kind == "begin":
        return {"kind": kind, "case": case, "problem": _problem(case, seed)}
    if kind == "batch":
        sims = [_sim(p) for p in _members(case, seed)]
        b = sim.Batch(len(sims))
        b.set(sims)
        return {"kind": kind, "case": case, "sims": sims, "batch": b}
    if kind == "serve":
        requests = []
        for k, p in enumerate(_members(case, seed)):
            wl = workloads.Workload("request %d" % k, p["lattice"], p["dims"], p["tau"],
                                    p["rho"].cpu().numpy(), p["u"].cpu().numpy(),
                                    p["theta"].cpu().numpy(), p["force"],
                                    _request_steps(case, k))
            requests.append(serve.Request(k, 0.0, wl, wl.steps))
        return {"kind": kind, "case": case, "requests": requests}
    s = _sim(_problem(case, seed))
    if kind == "restart":
        s.step(3)
        q = sim.Sim(s.lattice, s.dims, s.params.tau_hat, 1.0, 0.0, 1.0, storage=s.storage,
                    force_field=case["force"] == "field")
        _apply_force(q, _problem(case, seed))
        return {"kind": kind, "case": case, "sim": s, "into": q}
    return {"kind": kind, "case": case, "sim": s}


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def _values(populations, storage):
    """A checkpoint as numbers of the storage's own type."""
    return populations.view({"f64": torch.float64, "f32": torch.float32,
                             "f16dev": torch.float16}[storage])


def _snapshot(s):
    """The fields a program keeps: single precision where the storage is."""
    fields = s.moments()
    return fields if s.storage == "f64" else tuple(f.float() for f in fields)


def run(state):
    kind, case = state["kind"], state["case"]
    if kind == "begin":
        p = state["problem"]
        s = _sim(p)
        s.step(case["steps"])
        out = _snapshot(s)
        s.close()
        return out
    if kind == "batch":
        state["batch"].step(case["steps"])
        return [_snapshot(s) for s in state["sims"]]
    if kind == "serve":
        server = serve.Server(storage=case["storage"], max_slots=4, budget_bytes=4 << 30,
                              keep_populations=lambda rid: True)
        got = server.run(state["requests"], realtime=False)["results"]
        return [_values(r.populations, case["storage"])
                for r in sorted(got, key=lambda r: r.rid)]
    s = state["sim"]
    if kind == "restart":
        q = state["into"]
        saved = s.get_populations()
        q.set_populations(saved)
        q.step_count = s.step_count
        q.step(case["steps"])
        return _values(saved, s.storage), _values(q.get_populations(), s.storage)
    s.step(case["steps"])
    if kind == "watch":
        return [s.totals(), s.moments(), s.heat_flux()]
    if s.storage == "f16dev":
        return _values(s.get_populations(), s.storage)
    return _snapshot(s)


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def work(case):
    D = DIM[case["lattice"]]
    Q = 37 if D == 2 else 39
    s = BYTES[case["storage"]]
    kind = case["kind"]
    if kind in ("batch", "serve"):
        cells = [side * side for side in _sizes(case)]
        steps = [case["steps"] if kind == "batch" else _request_steps(case, k)
                 for k in range(len(cells))]
        out = 4 * (2 + D) if kind == "batch" and s == 4 else 8 * (2 + D) if kind == "batch" else 0
        each = [(2 * Q * s * n + (Q * s + out if kind == "batch" else 8 * (2 + D) + 2 * Q * s)) * c
                for c, n in zip(cells, steps)]
        return {"bytes": float(sum(each)),
                "flops": float(sum(15 * Q * n * c for c, n in zip(cells, steps)))}
    N = case["nx"] * case["ny"] * case["nz"]
    snapshot = Q * s + (2 + D) * (8 if case["storage"] == "f64" else 4)
    force = D * (8 if s == 8 else 4) if case["force"] == "field" else 0
    per = (2 * Q * s + force) * case["steps"]
    if kind == "begin":
        per += 8 * (2 + D) + Q * s + (8 * D if force else 0) + snapshot
    elif kind == "restart":
        per += 6 * Q * s
    elif kind == "watch":
        per += Q * s + 8 * (2 + 2 * D)  # the state read once for all three
    elif case["storage"] == "f16dev":
        per += 2 * Q * s
    else:
        per += snapshot
    return {"bytes": float(per) * N, "flops": float(15 * Q * case["steps"]) * N}


# ---------------------------------------------------------------------------
# the same in plain 64-bit arithmetic
# ---------------------------------------------------------------------------
# one velocity of each +c/-c pair, in the order of the population planes (the
# rest velocity first, then c and -c of each pair)
PAIRS = {
    "D2Q37": [(1, 0), (0, 1), (1, 1), (1, -1), (2, 0), (0, 2), (2, 1), (2, -1), (1, 2), (1, -2),
              (2, 2), (2, -2), (3, 0), (0, 3), (3, 1), (3, -1), (1, 3), (1, -3)],
    "D3Q39": [(1, 0, 0), (0, 1, 0), (0, 0, 1), (1, 1, 1), (1, 1, -1), (1, -1, 1), (1, -1, -1),
              (2, 0, 0), (0, 2, 0), (0, 0, 2), (2, 2, 0), (2, -2, 0), (2, 0, 2), (2, 0, -2),
              (0, 2, 2), (0, 2, -2), (3, 0, 0), (0, 3, 0), (0, 0, 3)],
}
# lattice scale of the Gauss-Hermite rule and the degree it integrates exactly
RULE = {"D2Q37": (1.1969797703930744, 9), "D3Q39": (math.sqrt(1.5), 7)}


def _rule(lattice):
    """Velocities (Q, D) as integers, their weights and the scale: the weights
    solve the Gaussian moment conditions, one weight a shell."""
    D = DIM[lattice]
    r, degree = RULE[lattice]
    c = [(0,) * D]
    for v in PAIRS[lattice]:
        c += [v, tuple(-k for k in v)]
    c = np.array(c)
    kinds = [tuple(sorted(abs(int(k)) for k in v)) for v in c]
    shells = sorted(set(kinds))
    xi = r * c.astype(np.longdouble)
    rows, want = [], []
    powers = [0, 2, 4, 6, 8]
    for a in np.ndindex(*(len(powers),) * D):
        e = [powers[k] for k in a]
        if sum(e) > degree:
            continue
        m = np.prod([xi[:, k] ** e[k] for k in range(D)], axis=0)
        rows.append([float(sum(m[i] for i in range(len(c)) if kinds[i] == s)) for s in shells])
        want.append(float(np.prod([math.prod(range(1, n, 2)) for n in e])))
    scale = np.abs(np.array(rows)).max(axis=1)
    w = np.linalg.lstsq(np.array(rows) / scale[:, None], np.array(want) / scale, rcond=None)[0]
    return c, np.array([w[shells.index(k)] for k in kinds]), r


class _Plain:
    """The model step by step in float64: populations f~ as (Q, nz, ny, nx), the
    post-collision value at its own node, a few velocities at a time."""

    def __init__(self, p):
        self.p = p
        self.D = D = DIM[p["lattice"]]
        self.c, self.w, self.r = _rule(p["lattice"])
        self.Q = len(self.w)
        nx, ny, nz = p["dims"]
        self.shape = (nz, ny, nx)
        self.N = nx * ny * nz
        self.dev = p["rho"].device
        kw = {"dtype": torch.float64, "device": self.dev}
        self.xi = torch.tensor(self.r * self.c, **kw)
        self.wt = torch.tensor(self.w, **kw)
        self.block = max(1, (1 << 25) // self.N)
        kind = p["force"][0]
        if kind == "uniform":
            g = torch.tensor(np.asarray(p["force"][1])[:D], **kw)[:, None].expand(D, self.N)
        elif kind == "axis":
            prof = torch.tensor(p["force"][2], **kw)
            at = [None, None, None]
            at[2 - p["force"][1]] = slice(None)
            g = torch.stack([prof[a][tuple(at)].expand(self.shape).reshape(-1) for a in range(D)])
        else:
            g = p["force"][1].reshape(D, self.N)
        self.g = g.to(self.dev)
        self.order = 4 if D == 2 else 3
        if p["walls"] is not None:
            tb, tt, ub, ut = p["walls"]
            self.emit = []
            for th, uw in ((tb, ub), (tt, ut)):
                u = torch.zeros((D, 1), **kw)
                u[0] = uw
                one = torch.ones(1, **kw)
                self.emit.append(self.equilibrium(slice(0, self.Q), one, u, th * one)[:, 0])
        tau = p["tau"]
        self.om, self.cf = 1.0 / tau, 1.0 - 0.5 / tau
        f = self.f0F(p["rho"], p["u"], p["theta"], None)
        self.A = torch.empty((self.Q,) + self.shape, **kw)
        for i in range(self.Q):
            fi = f[i].reshape(self.shape)
            self.A[i] = torch.roll(fi, [-k for k in self.shift(i)], (0, 1, 2))
            if p["walls"] is not None:
                for y in range(ny):
                    if not 0 <= y + self.c[i][1] < ny:
                        self.A[i, :, y] = fi[:, y]

    def shift(self, i):
        c = [int(k) for k in self.c[i]] + [0]
        return [c[2], c[1], c[0]]

    def blocks(self):
        return [slice(i, min(self.Q, i + self.block)) for i in range(0, self.Q, self.block)]

    def dot(self, s, v):
        return sum(self.xi[s, a][:, None] * v[a][None] for a in range(self.D))

    def equilibrium(self, s, rho, u, th):
        D = self.D
        X2 = (self.xi[s] ** 2).sum(1)[:, None]
        xu, u2, t = self.dot(s, u), (u * u).sum(0)[None], (th - 1)[None]
        e = 1 + xu + (xu ** 2 - u2 + t * (X2 - D)) / 2
        e = e + xu * (xu ** 2 - 3 * u2 + 3 * t * (X2 - D - 2)) / 6
        if self.order == 4:
            e = e + (xu ** 4 - 6 * xu ** 2 * u2 + 3 * u2 ** 2
                     + 6 * t * (xu ** 2 * (X2 - D - 4) + u2 * (D + 2 - X2))
                     + 3 * t ** 2 * (X2 ** 2 - 2 * (D + 2) * X2 + D * (D + 2))) / 24
        return self.wt[s][:, None] * rho[None] * e

    def force(self, s, rho, u, th, sig):
        D, g = self.D, self.g
        X2 = (self.xi[s] ** 2).sum(1)[:, None]
        xu, xg = self.dot(s, u), self.dot(s, g)
        u2, gu, t = (u * u).sum(0)[None], (u * g).sum(0)[None], (th - 1)[None]
        F = xg + xg * xu - gu + xg * (xu ** 2 - u2 + t * (X2 - D - 2)) / 2 - gu * xu
        F = F * rho[None]
        if sig is not None:
            sx = [sum(sig[a][b][None] * self.xi[s, b][:, None] for b in range(D))
                  for a in range(D)]
            F = F - (xg * sum(self.xi[s, a][:, None] * sx[a] for a in range(D))
                     - 2 * sum(sx[a] * g[a][None] for a in range(D))) / 2
        return self.wt[s][:, None] * F

    def f0F(self, rho, u, th, sig):
        f = torch.empty((self.Q, self.N), dtype=torch.float64, device=self.dev)
        for s in self.blocks():
            f[s] = self.equilibrium(s, rho, u, th) - 0.5 * self.force(s, rho, u, th, sig)
        return f

    def stream(self):
        f = torch.empty_like(self.A)
        for i in range(self.Q):
            f[i] = torch.roll(self.A[i], self.shift(i), (0, 1, 2))
        if self.p["walls"] is None:
            return f.reshape(self.Q, self.N)
        ny = self.shape[1]
        for side in (0, 1):
            absorbed = torch.zeros((self.shape[0], self.shape[2]), dtype=torch.float64,
                                   device=self.dev)
            norm = 0.0
            for i in range(self.Q):
                cy = int(self.c[i][1])
                if (cy > 0) == (side == 0) and cy != 0:
                    norm = norm + min(abs(cy), ny) * self.emit[side][i]
                for y in range(ny):
                    if (y + cy < 0) if side == 0 else (y + cy >= ny):
                        absorbed += self.A[i, :, y]
            rw = absorbed / norm
            for i in range(self.Q):
                cx, cy = int(self.c[i][0]), int(self.c[i][1])
                for y in range(ny):
                    if (y - cy < 0) if side == 0 else (y - cy >= ny):
                        f[i, :, y] = torch.roll(rw, cx, 1) * self.emit[side][i]
        return f.reshape(self.Q, self.N)

    def state(self, f):
        """rho, u, theta, the relaxation coefficients and the stress of f~."""
        D = self.D
        rho = f.sum(0)
        j = [self.block_sum(f, self.xi[:, a]) for a in range(D)]
        P = [[None] * D for _ in range(D)]
        for a in range(D):
            for b in range(a, D):
                P[a][b] = P[b][a] = self.block_sum(f, self.xi[:, a] * self.xi[:, b])
        ut = torch.stack([v / rho for v in j])
        u = ut + 0.5 * self.g
        E = sum(P[a][a] for a in range(D))
        th = (E / rho - (ut * ut).sum(0) + 0.25 * (self.g * self.g).sum(0)) / D
        om, cf = self.om, self.cf
        if self.p["mu"] > 0:
            om = 1.0 / (self.p["mu"] / (rho * th) + 0.5)
            cf = 1.0 - 0.5 * om
        g = self.g
        sig = [[-cf * (P[a][b] - rho * (u[a] * u[b] + (th if a == b else 0.0))
                       + 0.5 * rho * (u[a] * g[b] + g[a] * u[b])) for b in range(D)]
               for a in range(D)]
        tr = sum(sig[a][a] for a in range(D)) / D
        for a in range(D):
            sig[a][a] = sig[a][a] - tr
        return rho, u, th, om, cf, sig

    def block_sum(self, f, v):
        out = torch.zeros(self.N, dtype=torch.float64, device=self.dev)
        for s in self.blocks():
            out += (v[s][:, None] * f[s]).sum(0)
        return out

    def step(self, n):
        for _ in range(n):
            f = self.stream()
            rho, u, th, om, cf, sig = self.state(f)
            for s in self.blocks():
                f[s] += om * (self.equilibrium(s, rho, u, th) - f[s])
                f[s] += cf * self.force(s, rho, u, th, sig)
            self.A = f.reshape((self.Q,) + self.shape)

    def moments(self):
        rho, u, th = self.state(self.stream())[:3]
        return rho, u, th

    def totals(self):
        f = self.A.reshape(self.Q, self.N)
        m = f.sum(1)
        return np.array([float(m.sum())]
                        + [float((self.xi[:, a] * m).sum()) for a in range(self.D)]
                        + [float(((self.xi ** 2).sum(1) * m).sum())])

    def heat_flux(self):
        f = self.stream()
        rho, u, th, om, cf, sig = self.state(f)
        q = torch.zeros((self.D, self.N), dtype=torch.float64, device=self.dev)
        for s in self.blocks():
            f0 = self.equilibrium(s, rho, u, th)
            phys = f0 + cf * (f[s] - f0 + 0.5 * self.force(s, rho, u, th, sig))
            v = [self.xi[s, a][:, None] - u[a][None] for a in range(self.D)]
            e = 0.5 * phys * sum(k * k for k in v)
            for a in range(self.D):
                q[a] += (e * v[a]).sum(0)
        return q

    def populations(self):
        h = self.A.reshape(self.Q, self.N) - self.wt[:, None]
        if self.p["storage"] == "f16dev":
            h = h * (2.0 ** torch.round(-torch.log2(self.wt)))[:, None]
        return h.reshape(-1)


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        out = []
        for p in _members(case, seed):
            m = _Plain(p)
            m.step(case["steps"])
            out.append(m.moments())
        return out
    if kind == "serve":
        out = []
        for k, p in enumerate(_members(case, seed)):
            m = _Plain(p)
            m.step(_request_steps(case, k))
            out.append(m.populations().cpu())
        return out
    m = _Plain(_problem(case, seed))
    if kind == "restart":
        m.step(3)
        saved = m.populations()
        m.step(case["steps"])
        return saved, m.populations()
    m.step(case["steps"])
    if kind == "watch":
        return [m.totals(), m.moments(), m.heat_flux()]
    return m.populations() if case["storage"] == "f16dev" else m.moments()
