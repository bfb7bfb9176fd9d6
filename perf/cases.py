"""The work a user has this package do, as measurable cases.

A case is a plain dict.  `prepare` builds the run a program holds (parameters,
workspace, initial state, a checkpoint to restart from), `run` is one pass of
it through the public entry points (advance some steps, then read what the
program reads at that point), `exact` gives the same answers from a dense
64-bit torch form of the method, and `draw` makes further cases of the same
ranges.  Steps are read and written back in the storage precision of the run:
answers are kept in that precision too (a run that stores its fluid in FP16
does not know its sphere's force to more digits).

Keys of a case: `kind` picks the physical set-up, `prec` the storage
precision, `steps` the steps of a pass, `read` what is read after them.
"""
import math

import numpy as np
import torch

from paper_1909_01092_amd import workloads

Q = 19
MRT = {"tau_shear": 0.8, "tau_bulk": 1.1, "tau_mom": 0.9, "tau_ghost": 1.3}
KEEP = {"fp64": np.float64, "fp32": np.float32, "fp16": np.float16}
SIZE = {"fp64": 8, "fp32": 4, "fp16": 2}
RENEW = 1000  # steps after which a pass starts again from the checkpoint


# ------------------------------------------------------------------- cases
def listed():
    return [
        # a live view of a small channel: every step is looked at, so launches
        # and the round trip of one query are the whole cost
        dict(name="view_small_fp32", kind="channel", prec="fp32", nx=16, ny=16, nz=32, radius=3.0, kT=1e-5,
             steps=1, read="state"),
        # the double-precision reference run (24 x 24 x 48), whole populations saved
        dict(name="reference_fp64", kind="channel", prec="fp64", nx=24, ny=24, nz=48, radius=4.0, kT=1e-5,
             steps=100, read="populations"),
        # several spheres per fluid, batched: fluids with three, two and one sphere
        dict(name="spheres_fp32", kind="spheres", prec="fp32", nx=16, ny=16, nz=48, replicas=6, kT=1e-5,
             steps=40, read="state"),
        # distinct relaxation times in double precision, periodic box, no sphere
        dict(name="mrt_fluid_fp64", kind="box", prec="fp64", nx=50, ny=46, nz=130, walls=0, radius=0.0, kT=1e-4,
             mrt=True, steps=20, read="fields"),
        # confinement friction study: six radii, no noise, replayed as HIP graphs
        dict(name="friction_fp32", kind="friction", prec="fp32", nx=32, ny=32, nz=128, steps=80, graph=40,
             read="series"),
        # contact-angle study: nine wetting offsets in demixed closed boxes, no noise
        dict(name="wetting_fp32", kind="wetting", prec="fp32", nx=48, ny=48, nz=48, replicas=9, steps=50,
             read="state"),
        # one production channel, sampled for its flow profile
        dict(name="single_fp32", kind="channel", prec="fp32", nx=64, ny=64, nz=256, radius=8.0, kT=1e-5,
             steps=100, read="profile"),
        # the paper's closed 60 x 60 x 900 box and mixture
        dict(name="paper_box_fp32", kind="paper", prec="fp32", nx=60, ny=60, nz=900, radius=8.0, kT=1e-4,
             steps=50, read="profile"),
        # the batched ensemble: 192 replicas of three sizes, launch shape tuned once
        dict(name="ensemble_fp32", kind="ensemble", prec="fp32", replicas=192, kT=1e-5, steps=20, tune=8,
             read="state"),
        # the largest single channel, FP16 storage, launch shape tuned once
        dict(name="large_fp16", kind="channel", prec="fp16", nx=192, ny=192, nz=1024, radius=16.0, kT=1e-4,
             steps=15, tune=8, read="profile"),
        # gradient of the settling velocity on the adjoint channel (forward and reverse sweep)
        dict(name="adjoint_fp32", kind="channel", prec="fp32", nx=48, ny=48, nz=192, radius=6.0, kT=1e-5,
             steps=100, segment=50, read="adjoint"),
        # one iteration of a small fit through autograd: a fresh run, J and its gradient
        dict(name="fit_small_fp64", kind="channel", prec="fp64", nx=24, ny=24, nz=48, radius=4.0, kT=1e-5,
             steps=20, segment=10, read="autograd"),
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case: cross-sections of 12 to 192 nodes and lengths of 24 to
    1024, odd ones among them, each wall mask, storage, noise and relaxation."""
    prec = rng.choice(("fp32", "fp32", "fp64", "fp16"))
    grad = prec != "fp16" and rng.random() < 0.2
    nx, ny = _log(rng, 12, 96 if grad else 192), _log(rng, 12, 96 if grad else 192)
    nz = _log(rng, 24, 256 if grad else 1024)
    while nx * ny * nz > (6_000_000 if not grad else 800_000):
        nz = max(24, nz // 2)
        if nz == 24:
            nx, ny = max(12, nx * 2 // 3), max(12, ny * 2 // 3)
    N = nx * ny * nz
    rmax = (min(nx, ny, nz) - 7) / 2.0
    radius = round(rng.uniform(2.0, min(rmax, 12.0)), 2) if rmax > 2.2 and (grad or rng.random() < 0.85) else 0.0
    case = dict(kind="box", prec=prec, nx=nx, ny=ny, nz=nz, walls=rng.choice((3, 3, 7, 0, 1, 4)), radius=radius,
                kT=rng.choice((0.0, 1e-6, 1e-5, 1e-5, 1e-4)), drho=rng.choice((0.0, -0.1, 0.1)))
    if radius and not all(2 * math.ceil(radius) + 6 <= n for n in (nx, ny, nz)):
        case["walls"] = 7
    if grad:
        most = max(4, min(60, int(2e7 // N)))
        case.update(steps=rng.randint(4, most), segment=rng.choice((5, 20, 50)), read="adjoint", drho=0.1)
        return case
    if rng.random() < 0.25:
        case["mrt"] = True
    if rng.random() < 0.4:
        case["replicas"] = _log(rng, 2, max(2, min(64, int(6_000_000 // N))))
    case["steps"] = _log(rng, 5 if prec == "fp16" else 1, max(5, min(200, int(1.5e8 // (N * case.get("replicas", 1))))))
    small = N * case.get("replicas", 1) < 400_000
    case["read"] = rng.choice(("state", "series", "profile", "fields", "populations") if small else
                              ("state", "series", "profile"))
    if case["read"] in ("state", "series") and not radius:
        case["read"] = "profile"
    return case


# ------------------------------------------------------------------- inputs
def _replicas(case, seed):
    """Parameter sets of a case.  The seed sets the noise, the initial density
    noise and where in its cell each sphere starts."""
    rng = np.random.default_rng(seed)
    kind, nrep = case["kind"], int(case.get("replicas", 1))
    key = int(rng.integers(1, 1 << 40))

    def off():
        return rng.uniform(-0.45, 0.45, 3)

    def at(p, c=None):
        c = [(p[k] - 1) / 2.0 for k in ("nx", "ny", "nz")] if c is None else c
        return tuple(float(a + d) for a, d in zip(c, off()))

    if kind == "ensemble":
        reps = workloads.ensemble(steps_cap=256)
        step = max(1, len(reps) // nrep)
        reps = [dict(p, seed=key, kT=case["kT"], X0=at(p)) for p in reps[::step][:nrep]]
    elif kind == "friction":
        reps = [dict(p, seed=key, X0=at(p)) for p in workloads.friction(steps_cap=256)]
    elif kind == "wetting":
        reps = [dict(p, seed=key, X0=at(p)) for p in workloads.wetting(n=case["nx"], steps_cap=256)[:nrep]]
    elif kind == "paper":
        p = workloads.paper_box(n=case["nx"], nz=case["nz"], radius=case["radius"], kT=case["kT"], steps_cap=256)
        reps = [dict(p, seed=key, X0=at(p, p["X0"]))]
    elif kind == "spheres":
        reps = []
        for r in range(nrep):
            p = workloads.full(dict(nx=case["nx"], ny=case["ny"], nz=case["nz"], walls=0, init_amp=1e-3, G=1.2,
                                    kT=case["kT"], g=(0.0, 0.0, 1e-4), seed=key, replica=r, radius=2.5, wet_drho=0.1,
                                    series_cap=256))
            c = [(p["nx"] - 1) / 2.0, (p["ny"] - 1) / 2.0]
            p["X0"] = at(p, c + [p["nz"] / 6.0])
            p["spheres"] = [dict(radius=2.1 + 0.3 * k, rho_p=2.0, wet_drho=0.1 * (k - 0.5),
                                 X0=at(p, c + [p["nz"] * (3 + 2 * k) / 6.0])) for k in range(2 - r % 3)]
            reps.append(p)
    else:  # a channel at the workloads' parameters, or a box of any walls
        g = (0.0, 0.0, {192: 1e-4, 64: 1e-4}.get(case["nx"], 5e-5) if kind == "channel" else 1e-5)
        reps = []
        for r in range(nrep):
            p = workloads.full(dict(nx=case["nx"], ny=case["ny"], nz=case["nz"], walls=case.get("walls", 3),
                                    init_amp=1e-3, G=1.5, rho_p=2.0, kT=case["kT"], radius=case["radius"], g=g,
                                    wet_drho=case.get("drho", 0.0), seed=key, replica=r, series_cap=256))
            reps.append(dict(p, X0=at(p)) if p["radius"] else p)
    if case.get("mrt"):
        reps = [dict(p, **MRT) for p in reps]
    return reps


def prepare(case, seed):
    from paper_1909_01092_amd.sim import Simulation
    reps = _replicas(case, seed)
    state = dict(case=case, reps=reps, keep=KEEP[case["prec"]], done=0)
    if case["read"] == "autograd":
        p = reps[0]
        state["theta"] = torch.tensor([*p["g"], p["G"], p["wet_drho"]], dtype=torch.float64, requires_grad=True)
        return state
    sim = Simulation(reps, precision=case["prec"], stream=torch.cuda.Stream() if case.get("graph") else None)
    if case.get("tune"):
        sim.autotune(steps_per_trial=case["tune"], preserve=True)
    if case.get("graph"):
        sim.set_graph(case["graph"])
    state.update(sim=sim, start=sim.checkpoint())
    return state


def _entries(reps):
    """(first entry index, number of entries) of each replica."""
    at, out = 0, []
    for p in reps:
        n = 1 + len(p.get("spheres", ()))
        out.append((at, n))
        at += n
    return out


def _vectors(case):
    """The sphere's vectors that are read (W and delta lie below FP16's range)."""
    return ("X", "U", "F") if case["prec"] == "fp16" else ("X", "U", "W", "F", "delta")


def run(state):
    case, keep = state["case"], state["keep"]
    steps, read = case["steps"], case["read"]
    if read == "autograd":
        from paper_1909_01092_amd.autograd import settling_velocity
        theta = state["theta"]
        theta.grad = None
        J = settling_velocity(theta, state["reps"][0], steps, case["prec"], case["segment"])
        J.backward()
        return {"J": J.detach(), "grad": theta.grad}
    sim = state["sim"]
    if state["done"] + steps > RENEW:  # a long program starts over
        sim.restore(state["start"])
        state["done"] = 0
    state["done"] += steps
    if read == "adjoint":
        J, grad = sim.adjoint(steps, case["segment"])
        return {"J": keep(J), "grad": grad.astype(keep)}
    sim.step(steps)
    ent = _entries(state["reps"])
    out = {}
    if any(p["radius"] > 0 for p in state["reps"]):
        balls = [sim.particle_state(e) for at, n in ent for e in range(at, at + n)]
        for key in _vectors(case):
            out[key] = np.stack([b[key] for b in balls]).astype(keep)
        for key in ("step", "n_covered", "n_uncovered", "n_links"):
            out[key] = np.array([b[key] for b in balls])
    if read == "series":
        out["series"] = np.stack([sim.u_series(e)[-steps:] for at, n in ent for e in range(at, at + n)]).astype(keep)
    elif read == "profile":
        obs = [sim.observables(at, profile=True) for at, n in ent]
        out["mass"] = np.stack([o["mass"] for o in obs]).astype(np.float32 if keep is np.float16 else keep)
        out["profile"] = np.stack([o["uz_profile"] for o in obs]).astype(keep)
        out["u2"] = np.array([o["u2_mean"] for o in obs]).astype(keep)
    elif read == "fields":
        for k, (at, n) in enumerate(ent[:8]):
            rho, u = sim.fields(at)
            out["rho%d" % k], out["u%d" % k] = rho.astype(keep), u.astype(keep)
    elif read == "populations":
        for k, (at, n) in enumerate(ent[:8]):
            out["f%d" % k] = sim.populations(at).astype(keep)
    return out


def _nodes(case):
    if case["kind"] == "ensemble":
        reps = workloads.ensemble()
        reps = reps[::max(1, len(reps) // case["replicas"])][:case["replicas"]]
        return sum(p["nx"] * p["ny"] * p["nz"] for p in reps)
    n = case["nx"] * case["ny"] * case["nz"]
    return n * (len(workloads.FRICTION_RADII) if case["kind"] == "friction" else int(case.get("replicas", 1)))


def work(case):
    """Per step and node: 2 x 19 populations read once and written once; the
    sums, force, transforms and (with noise) 33 Box-Muller normals in flops.
    A reverse step reads and writes eight moment adjoints, reads the eight
    moments of the step, and takes about the flops of a forward one twice."""
    n = float(_nodes(case)) * case["steps"]
    noisy = case.get("kT", 0.0) > 0.0
    per_b, per_f = 2 * 38 * SIZE[case["prec"]], 700.0 + (300.0 if noisy else 0.0) + (600.0 if case.get("mrt") else 0.0)
    if case["read"] in ("adjoint", "autograd"):
        per_b += 24 * SIZE[case["prec"]]
        per_f *= 3.0
    return {"bytes": n * per_b, "flops": n * per_f}


# ------------------------------------------------------------------- exact
C = np.array([(0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1), (1, 1, 0), (-1, -1, 0),
              (1, -1, 0), (-1, 1, 0), (1, 0, 1), (-1, 0, -1), (1, 0, -1), (-1, 0, 1), (0, 1, 1), (0, -1, -1),
              (0, 1, -1), (0, -1, 1)])
WGT = np.array([1 / 3] + 6 * [1 / 18] + 12 * [1 / 36])
OPP = [int(np.flatnonzero((C == -c).all(1))[0]) for c in C]


def _basis():
    x, y, z = C.T.astype(float)
    c2 = x * x + y * y + z * z
    E = np.array([1 + 0 * x, x, y, z, c2 - 1, 3 * x * x - c2, y * y - z * z, x * y, y * z, x * z, (3 * c2 - 5) * x,
                  (3 * c2 - 5) * y, (3 * c2 - 5) * z, (y * y - z * z) * x, (z * z - x * x) * y, (x * x - y * y) * z,
                  3 * c2 * c2 - 6 * c2 + 1, (2 * c2 - 3) * (3 * x * x - c2), (2 * c2 - 3) * (y * y - z * z)])
    return E, (WGT * E * E).sum(1)


def _philox(c, k0, k1):
    """Philox4x32-10 on int64 tensors or ints holding 32-bit words."""
    m = 0xFFFFFFFF
    c0, c1, c2, c3 = c
    for _ in range(10):
        a, b = c0 * 0xD2511F53, c2 * 0xCD9E8D57  # tensors wrap at 64 bits: the low words stay right
        c0, c1, c2, c3 = ((b >> 32) & m) ^ c1 ^ k0, b & m, ((a >> 32) & m) ^ c3 ^ k1, a & m
        k0, k1 = (k0 + 0x9E3779B9) & m, (k1 + 0xBB67AE85) & m
    return c0, c1, c2, c3


class Dense:
    """One fluid with its spheres in 64 bits on whole arrays [.., z, y, x]."""

    def __init__(self, p, dev):
        self.p, self.dev = p, dev
        self.n = (p["nx"], p["ny"], p["nz"])
        self.wall = [bool(p["walls"] >> a & 1) for a in range(3)]
        E, b = _basis()
        self.E, self.b = torch.tensor(E, device=dev), torch.tensor(b, device=dev)
        self.back = torch.tensor(WGT[:, None] * E.T / b[None, :], device=dev)
        self.node = torch.arange(self.n[0] * self.n[1] * self.n[2], device=dev).reshape(self.n[::-1])
        ball = [p] + list(p.get("spheres", ())) if p["radius"] > 0 else []
        self.balls = [dict(R=float(s["radius"]), rho=float(s["rho_p"]), dr=float(s["wet_drho"]),
                           X=np.array(s["X0"], float), U=np.array(s.get("U0", (0, 0, 0)), float),
                           W=np.array(s.get("W0", (0, 0, 0)), float), F=np.zeros(3), T=np.zeros(3), Pev=np.zeros(3),
                           Lev=np.zeros(3), n_covered=0, n_uncovered=0, n_links=0) for s in ball]
        for s in self.balls:
            s["V"] = 4.0 / 3.0 * math.pi * s["R"] ** 3
        self.k = (p["seed"] & 0xFFFFFFFF, (p["seed"] >> 32) ^ p["replica"])
        self.step, self.delta, self.series = 0, np.zeros(2), []
        self.solid = self.owner()
        w = _philox((self.node, 0, 0, 1), *self.k)[:2]
        f = []
        for l in range(2):
            base = torch.full(self.n[::-1], float(p["rho0"][l]), dtype=torch.float64, device=dev)
            if p["init_split"] > 0:
                base[p["init_split"]:] = float(p["rho0"][1 - l])
            rho = base + p["init_amp"] * (2.0 * ((w[l].double() + 0.5) * 2.0 ** -32) - 1.0)
            rho[self.solid > 0] = 0.0
            f.append(torch.tensor(WGT, device=dev)[:, None, None, None] * rho)
        self.f = torch.stack(f)
        tot0 = p["rho0"][0] + p["rho0"][1]
        g = np.array(p["g"], float)
        for s in self.balls:
            s["Fext"] = s["V"] * (s["rho"] - tot0) * g
        self.af = -sum((s["Fext"] for s in self.balls), np.zeros(3)) / float(self.f.sum())

    # geometry
    def axes(self, X, half=(0.0, 0.0, 0.0)):
        """Minimum-image separations of the nodes (moved by `half`) from X."""
        out = []
        for a in range(3):
            d = torch.arange(self.n[a], dtype=torch.float64, device=self.dev) + half[a] - float(X[a])
            if not self.wall[a]:
                h = 0.5 * self.n[a]
                d = torch.where(d > h, d - self.n[a], torch.where(d < -h, d + self.n[a], d))
            out.append(d.reshape([-1 if b == 2 - a else 1 for b in range(3)]))
        return out

    def owner(self):
        own = torch.zeros(self.n[::-1], dtype=torch.int64, device=self.dev)
        for k, s in reversed(list(enumerate(self.balls))):
            x, y, z = self.axes(s["X"])
            own[(x * x + y * y) + z * z < s["R"] * s["R"]] = k + 1
        return own

    def at(self, A, c):
        """A at x + c: wrapped on periodic axes, the last node again beyond a wall."""
        i = []
        for a in range(3):
            v = torch.arange(self.n[a], device=self.dev) + int(c[a])
            i.append(v.clamp(0, self.n[a] - 1) if self.wall[a] else v % self.n[a])
        return A[..., i[2][:, None, None], i[1][None, :, None], i[0][None, None, :]]

    def inside(self, c):
        ok = torch.ones(self.n[::-1], dtype=torch.bool, device=self.dev)
        for a in range(3):
            if self.wall[a] and c[a]:
                i = [slice(None)] * 3
                i[2 - a] = self.n[a] - 1 if c[a] > 0 else 0
                ok[tuple(i)] = False
        return ok

    # one step
    def moments(self):
        m = torch.tensordot(self.E[:4], self.f, dims=([1], [1])).transpose(0, 1)
        return m[:, 0], m[:, 1:]

    def seen(self, rho):
        rt = rho.clone()
        if not self.balls:
            return rt
        s, cnt = torch.zeros_like(rho), torch.zeros_like(rho[0])
        for c in C[1:]:
            ok = self.inside(c) & (self.at(self.solid, c) == 0)
            s += torch.where(ok, self.at(rho, c), 0.0)
            cnt += ok
        for k, ball in enumerate(self.balls):
            m = self.solid == k + 1
            for l, sg in ((0, 1.0), (1, -1.0)):
                rt[l] = torch.where(m, torch.where(cnt > 0, s[l] / cnt.clamp(min=1) + sg * ball["dr"], 0.0), rt[l])
        return rt

    def force(self, rho):
        rt, G, fluid = self.seen(rho), self.p["G"], self.solid == 0
        F = torch.zeros((2, 3) + tuple(rho.shape[1:]), dtype=torch.float64, device=self.dev)
        self.react = [[np.zeros(3), np.zeros(3)] for _ in self.balls]
        for i in range(1, Q):
            there = self.at(rt, C[i])
            link = -G * WGT[i] * rho * there.flip(0) * fluid
            for a in range(3):
                if C[i][a]:
                    F[:, a] += link * int(C[i][a])
            for k, ball in enumerate(self.balls):
                m = self.inside(C[i]) & (self.at(self.solid, C[i]) == k + 1)
                self.add(self.react[k], link.sum(0) * m, i, ball)
        for a in range(3):
            F[:, a] += rho * float(self.af[a])
        return F

    def add(self, to, size, i, ball):
        """Force size * c_i at the link midpoints, and its torque about the ball, onto `to`."""
        r = self.axes(ball["X"], 0.5 * C[i])
        s = np.array([float(size.sum())] + [float((size * d).sum()) for d in r])
        to[0] += s[0] * C[i]
        to[1] += np.cross(s[1:], C[i])

    def noise(self):
        z = []
        for b in range(9):
            w = _philox((self.node, self.step, b, 0), *self.k)
            for h in (0, 2):
                u1, u2 = (w[h].double() + 0.5) * 2.0 ** -32, (w[h + 1].double() + 0.5) * 2.0 ** -32
                r, a = torch.sqrt(-2.0 * torch.log(u1)), 2.0 * math.pi * u2
                z += [r * torch.cos(a), r * torch.sin(a)]
        return z

    def collide(self, rho, j, F):
        p = self.p
        gs, gb, gj, gg = (1.0 - 1.0 / p[k] for k in ("tau_shear", "tau_bulk", "tau_mom", "tau_ghost"))
        mu, tot = 3.0 * p["kT"], rho.sum(0)
        u = (j.sum(0) + 0.5 * F.sum(0)) / torch.where(tot > 0, tot, 1.0)
        z = self.noise() if mu > 0 else None
        pos = rho.clamp(min=0.0)
        ux, uy, uz = u
        uu = ux * ux + uy * uy + uz * uz
        out = []
        for l, sg in ((0, 1.0), (1, -1.0)):
            r, Fl = rho[l], F[l]
            m = torch.tensordot(self.E, self.f[l], dims=([1], [0]))
            n = [m[0]]
            for a in range(3):
                v = r * u[a] + gj * (j[l, a] + 0.5 * Fl[a] - r * u[a]) + 0.5 * Fl[a]
                if mu > 0 and p["noise_diffusive"]:
                    amp = torch.sqrt(mu * float(self.b[1]) * (1 - gj * gj) * pos[0] * pos[1] / torch.where(tot > 0, tot, 1.0))
                    v = v + sg * amp * z[32 + a]
                n.append(v)
            uF = ux * Fl[0] + uy * Fl[1] + uz * Fl[2]
            eq = (r * uu, r * (3 * ux * ux - uu), r * (uy * uy - uz * uz), r * ux * uy, r * uy * uz, r * ux * uz)
            ph = (2 * uF, 2 * (3 * ux * Fl[0] - uF), 2 * (uy * Fl[1] - uz * Fl[2]), ux * Fl[1] + uy * Fl[0],
                  uy * Fl[2] + uz * Fl[1], ux * Fl[2] + uz * Fl[0])
            for k in range(4, Q):
                g = gb if k == 4 else gs if k < 10 else gg
                v = eq[k - 4] + g * (m[k] - eq[k - 4]) + 0.5 * (1 + g) * ph[k - 4] if k < 10 else g * m[k]
                if mu > 0:
                    v = v + torch.sqrt(mu * pos[l] * float(self.b[k]) * (1 - g * g)) * z[16 * l + k - 4]
                n.append(v)
            out.append(torch.tensordot(self.back, torch.stack(n), dims=([1], [0])))
        post = torch.stack(out)
        return post * (self.solid == 0)

    def advance(self):
        p, fluid = self.p, self.solid == 0
        rho, j = self.moments()
        F = self.force(rho)
        post = self.collide(rho, j, F)
        new, dm = post.clone(), np.zeros(2)
        push = [[np.zeros(3), np.zeros(3)] for _ in self.balls]
        for s in self.balls:
            s["n_links"] = 0
        for i in range(1, Q):
            o, c = OPP[i], -C[i]  # population i arrives from x + c; a link there points along c
            src, own = self.at(post[:, i], c), self.at(self.solid, c)
            ok = self.inside(c)
            got = torch.where(ok, src, post[:, o])
            for k, s in enumerate(self.balls):
                m = ok & (own == k + 1) & fluid
                cnt = int(m.sum())
                if not cnt:
                    continue
                s["n_links"] += cnt
                x, y, z = self.axes(s["X"], 0.5 * c)
                W, U = s["W"], s["U"]
                cu = (float(c @ U) + (W[1] * z - W[2] * y) * int(c[0]) + (W[2] * x - W[0] * z) * int(c[1])
                      + (W[0] * y - W[1] * x) * int(c[2]))
                corr = 6.0 * WGT[i] * rho * cu
                got = torch.where(m, post[:, o] - corr, got)
                self.add(push[k], (2.0 * post[:, o] - corr).sum(0) * m, o, s)
                dm -= (corr * m).sum((1, 2, 3)).cpu().numpy()
            new[:, i] = got
        new *= fluid
        for k, s in enumerate(self.balls):
            mass = s["rho"] * s["V"]
            s["F"] = push[k][0] - self.react[k][0] + s["Fext"] + s["Pev"]
            s["T"] = push[k][1] - self.react[k][1] + s["Lev"]
            s["U"] = s["U"] + s["F"] / mass
            s["W"] = s["W"] + s["T"] / (0.4 * mass * s["R"] ** 2)
            s["X"] = s["X"] + s["U"]
            for a in range(3):
                if not self.wall[a]:
                    s["X"][a] += self.n[a] if s["X"][a] < 0 else -self.n[a] if s["X"][a] >= self.n[a] else 0.0
            s["Pev"], s["Lev"] = np.zeros(3), np.zeros(3)
        self.series.append([s["U"].copy() for s in self.balls])
        if self.balls:
            self.events(new, dm)
        self.f, self.step = new, self.step + 1

    def events(self, new, dm):
        was, now = self.solid, self.owner()
        m = torch.tensordot(self.E[:4], new, dims=([1], [1])).transpose(0, 1)
        rho, jt = m[:, 0], m[:, 1:].sum(0)
        for q in torch.nonzero((was == 0) & (now > 0)).tolist():
            s = self.balls[int(now[tuple(q)]) - 1]
            r = self.from_centre(q, s)
            v = jt[(slice(None),) + tuple(q)].cpu().numpy()
            s["Pev"] += v
            s["Lev"] += np.cross(r, v)
            s["n_covered"] += 1
            dm -= rho[(slice(None),) + tuple(q)].cpu().numpy()
        for q in torch.nonzero((was > 0) & (now == 0)).tolist():
            s = self.balls[int(was[tuple(q)]) - 1]
            got = []
            for c in C[1:]:
                w = [q[2] + int(c[0]), q[1] + int(c[1]), q[0] + int(c[2])]
                if any(self.wall[a] and not 0 <= w[a] < self.n[a] for a in range(3)):
                    continue
                w = tuple(w[a] % self.n[a] for a in (2, 1, 0))
                if not int(was[w]) and not int(now[w]):
                    got.append(rho[(slice(None),) + w].cpu().numpy())
            rb = np.mean(got, 0) if got else np.array(self.p["rho0"], float)
            r = self.from_centre(q, s)
            u = s["U"] + np.cross(s["W"], r)
            cu = C @ u
            eq = WGT * (1.0 + 3.0 * cu + 4.5 * cu * cu - 1.5 * (u @ u))
            new[(slice(None), slice(None)) + tuple(q)] = torch.tensor(rb[:, None] * eq, device=self.dev)
            dm += rb
            s["Pev"] -= rb.sum() * u
            s["Lev"] -= np.cross(r, rb.sum() * u)
            s["n_uncovered"] += 1
        new *= now == 0
        self.delta = -dm / float((now == 0).sum())
        new += (torch.tensor(WGT[None, :] * self.delta[:, None], device=self.dev)[:, :, None, None, None]) * (now == 0)
        self.solid = now

    def from_centre(self, q, s):
        return np.array([float(d.flatten()[q[2 - a]]) for a, d in enumerate(self.axes(s["X"]))])

    def velocity(self):
        rho, j = self.moments()
        tot = rho.sum(0)
        F = self.force(rho)
        return rho, (j.sum(0) + 0.5 * F.sum(0)) / torch.where(tot > 0, tot, 1.0) * (self.solid == 0)


def _seconds(case, reps):
    """About what `exact` takes for a case on the GPU."""
    n = sum(p["nx"] * p["ny"] * p["nz"] for p in reps)
    links = sum(1 + len(p.get("spheres", ())) for p in reps)
    return case["steps"] * (0.03 * links + n * 2.8e-8)


def exact(case, seed):
    reps, steps, read = _replicas(case, seed), case["steps"], case["read"]
    if _seconds(case, reps) > 18.0:
        return None
    dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
    out, balls, series = {}, [], []
    mass, prof, u2 = [], [], []
    for k, p in enumerate(reps):
        d = Dense(p, dev)
        for _ in range(steps):
            d.advance()
        balls += [dict(s, delta=d.delta, step=d.step) for s in d.balls]
        series += [[s[b] for s in d.series] for b in range(len(d.balls))]
        if read in ("profile", "fields"):
            rho, u = d.velocity()
            fluid = (d.solid == 0).double()
            if read == "fields" and k < 8:
                out["rho%d" % k], out["u%d" % k] = rho, u
            mass.append(rho.sum((1, 2, 3)).cpu().numpy())
            prof.append((u[2].sum(0) / fluid.sum(0).clamp(min=1)).cpu().numpy())
            u2.append(float((u * u).sum() / fluid.sum()))
        elif read == "populations" and k < 8:
            out["f%d" % k] = d.f
    if read in ("adjoint", "autograd"):
        J = float(np.mean([s[2] for s in series[0]]))
        return {"J": np.float64(J), "grad": None}
    if balls:
        for key in _vectors(case):
            out[key] = np.stack([b[key] for b in balls])
        for key in ("step", "n_covered", "n_uncovered", "n_links"):
            out[key] = np.array([b[key] for b in balls])
    if read == "series":
        out["series"] = np.array(series)
    elif read == "profile":
        out["mass"], out["profile"], out["u2"] = np.stack(mass), np.stack(prof), np.array(u2)
    return out
