"""Performance cases of the lattice Boltzmann library: what its users run.

A case is one pass through the public entry points of ``paper_1406_2211_amd``
as a simulation program makes it: a number of time steps of one box followed by
the output of that program's frame (velocity and density field, particle
state), a steady batch of ensemble boxes, or a whole serving call.  Boxes of
FP64 storage write FP64 frames, the others single-precision ones.

``exact`` computes the same pass in 64 bits with plain torch operations: the
unfused operator sequence (half force, collision, streaming, half force) with
the coupling of the paper's Sec. 5 and 6.
"""
import math

import numpy as np
import torch

from paper_1406_2211_amd import inputs as I
from paper_1406_2211_amd import lbc as L
from paper_1406_2211_amd import serving as S

STORAGE = {"f64": L.LB_F64, "f32": L.LB_F32, "f16": L.LB_F16, "bf16": L.LB_BF16}
STORED_BYTES = {"f64": 8, "f32": 4, "f16": 2, "bf16": 2}
COLLISION = {"bgk": L.LB_BGK, "trt": L.LB_TRT, "mrt": L.LB_MRT}
COUPLING = {"none": L.LB_COUPLE_NONE, "fc": L.LB_COUPLE_FC, "ebf": L.LB_COUPLE_EBF,
            "ib": L.LB_COUPLE_IB}
MRT_RATES = (1.4, 1.2, 1.2, 1.5, 1.5)
F16_SCALE = 20   # stored deviations of these flows stay below about 5e-3
MAGIC = 3.0 / 16.0
FLOPS_PER_SITE = 250.0   # moments, equilibria and relaxation of one D3Q19 site


def _box(**kw):
    """A single-box case with the defaults of a plain force-coupled run."""
    c = dict(kind="box", nx=32, ny=32, nz=32, wall=False, storage="f32", collision="bgk",
             coupling="fc", kernel=2, tau=0.8, force=0.0, gamma=1.0, particles=0, chains=0,
             beads=0, substeps=0, inside=False, shells=0, subdivisions=0, radius=0.0, kT=0.0,
             deterministic=False, steps=10, frame="fluid")
    c.update(kw)
    return c


def listed():
    return [
        # the smallest run: one tracer in a 32^3 box, every launch shows
        _box(name="single_particle_32_f64", storage="f64", particles=1, steps=10),
        # a small walled channel of ragged size, read after every step by the
        # program that steers it
        _box(name="steered_channel_odd", nx=45, ny=37, nz=52, wall=True, force=1e-6, kernel=3,
             particles=200, steps=1),
        # an ordinary suspension of free particles, one per hundred sites
        _box(name="suspension_128", nx=128, ny=128, nz=128, collision="trt", tau=0.6, gamma=2.0,
             particles=20000, steps=10),
        # polymer chains with the coupling inside every sub-step
        _box(name="chains_inside_128", nx=128, ny=128, nz=128, collision="trt", tau=0.6,
             gamma=2.0, chains=12, beads=100, substeps=5, inside=True, steps=10),
        # the large polymer solution of the benchmark, and its 16-bit form
        _box(name="chains_256", nx=256, ny=256, nz=256, collision="trt", tau=0.6, gamma=2.0,
             chains=100, beads=100, substeps=5, steps=10),
        _box(name="chains_256_f16", nx=256, ny=256, nz=256, storage="f16", collision="trt",
             tau=0.6, gamma=2.0, chains=100, beads=100, substeps=5, steps=10),
        # the immersed-boundary channel of the benchmark: 64 shells, four-point kernel
        _box(name="shell_channel", nx=128, ny=128, nz=256, wall=True, force=1e-6, coupling="ib",
             kernel=4, shells=64, subdivisions=3, radius=6.0, steps=10),
        # a few shells in a small periodic box of odd size, FP64, three-point kernel
        _box(name="few_shells_odd_f64", nx=72, ny=60, nz=75, storage="f64", coupling="ib",
             kernel=3, shells=4, subdivisions=2, radius=5.0, steps=10),
        # fluctuating fluid with the random coupling force
        _box(name="thermal_192", nx=192, ny=192, nz=192, collision="trt", tau=0.6, gamma=2.0,
             particles=5000, kT=1e-5, steps=10),
        # general MRT collision on a ragged box, and every field written out
        # (analysis of a run)
        _box(name="mrt_odd_analysis", nx=150, ny=117, nz=133, collision="mrt", tau=0.6,
             coupling="ebf", gamma=2.0, particles=2000, steps=10, frame="all"),
        # uneven boxes advanced together, between two admissions of a server
        dict(name="ensemble_24", kind="ensemble", boxes=24, mix=5, storage="f16", low=32, high=160,
             most_particles=5000, steps=20),
        # a whole serving call: admission, batched steps, results
        dict(name="serving_24", kind="serving", boxes=24, mix=5, low=32, high=160,
             most_particles=5000, low_steps=40, high_steps=120),
    ]


def _log_uniform(rng, low, high):
    return int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))


def _sides(rng, low, high, most):
    """Three box sides, log-uniform, with at most `most` sites; half of them odd or even as they
    fall, half a multiple of 32 as users like to choose them."""
    while True:
        n = [_log_uniform(rng, low, high) for _ in range(3)]
        if rng.random() < 0.5:
            n = [max(32, (k + 16) // 32 * 32) for k in n]
        if n[0] * n[1] * n[2] <= most:
            return dict(nx=n[0], ny=n[1], nz=n[2])


def draw(rng):
    kind = rng.choice(["free", "free", "chains", "shells", "ensemble", "serving"])
    if kind == "ensemble":
        return dict(kind="ensemble", boxes=rng.randint(4, 24), mix=rng.randint(1, 99),
                    storage=rng.choice(["f16", "f32"]), low=24, high=rng.randint(64, 150),
                    most_particles=rng.randint(200, 5000), steps=rng.randint(5, 20))
    if kind == "serving":
        return dict(kind="serving", boxes=rng.randint(6, 24), mix=rng.randint(1, 99),
                    low=32, high=rng.randint(80, 160),
                    most_particles=rng.randint(500, 5000), low_steps=20,
                    high_steps=rng.randint(40, 120))
    if kind == "shells":
        c = _box(**_sides(rng, 48, 160, 1 << 22), coupling="ib", kernel=rng.choice([2, 3, 4]),
                 wall=rng.random() < 0.5, storage=rng.choice(["f32", "f32", "f64"]),
                 subdivisions=rng.choice([2, 3]), radius=rng.choice([4.0, 5.0, 6.0]),
                 steps=rng.randint(2, 10))
        room = c["nx"] * c["ny"] * c["nz"] / (2 * c["radius"] + 6) ** 3
        c["shells"] = max(1, min(64, int(room * rng.uniform(0.05, 0.25))))
        if c["wall"]:
            c["force"] = 1e-6
        return c
    if kind == "chains":
        c = _box(**_sides(rng, 40, 220, 1 << 23), collision=rng.choice(["trt", "bgk"]), tau=0.6,
                 gamma=2.0, storage=rng.choice(["f32", "f32", "f16", "f64"]),
                 beads=rng.randint(10, 120), substeps=rng.randint(3, 7),
                 inside=rng.random() < 0.5, steps=rng.randint(2, 10))
        c["chains"] = max(1, min(100, c["nx"] * c["ny"] * c["nz"] // (1600 * c["beads"])))
        return c
    c = _box(**_sides(rng, 24, 240, 1 << 23), collision=rng.choice(["bgk", "trt", "mrt"]),
             coupling=rng.choice(["fc", "fc", "ebf"]), kernel=rng.choice([2, 2, 3, 4]),
             storage=rng.choice(["f32", "f32", "f64", "f16", "bf16"]),
             wall=rng.random() < 0.3, tau=round(rng.uniform(0.6, 1.0), 3),
             deterministic=rng.random() < 0.1, steps=rng.randint(1, 10),
             frame=rng.choice(["fluid", "fluid", "all"]))
    c["particles"] = _log_uniform(rng, 1, max(2, min(20000, c["nx"] * c["ny"] * c["nz"] // 100)))
    if c["wall"]:
        c["force"] = 1e-6
    elif c["storage"] in ("f32", "f64") and rng.random() < 0.3:
        c["kT"] = 1e-5
    return c


# ------------------------------------------------------------------- inputs
def _flow(case, seed):
    """Smooth initial velocity [3, nz, ny, nx]: three random long waves per component of
    amplitude about 0.01 (vanishing mean), on the GPU."""
    g = np.random.default_rng(seed)
    dims = (case["nz"], case["ny"], case["nx"])
    u = torch.zeros((3,) + dims, dtype=torch.float64, device="cuda")
    for a in range(3):
        for _ in range(3):
            waves = []
            for axis, n in enumerate(dims):
                k, ph = int(g.integers(0, 3)), g.uniform(0.0, 2.0 * math.pi)
                x = torch.arange(n, dtype=torch.float64, device="cuda")
                waves.append(torch.cos(2.0 * math.pi * max(k, 1) / n * x + ph))
            u[a] += 0.006 * waves[0][:, None, None] * waves[1][None, :, None] * waves[2][None, None, :]
    return u


def _particles(case, seed):
    """Host arrays: positions, velocities, bonds, shell template (those the case has)."""
    box = (case["nx"], case["ny"], case["nz"])
    out = dict(pos=None, vel=None, bonds=None, template=None)
    if case["chains"]:
        out["pos"], out["vel"], out["bonds"] = I.chains(case["chains"], case["beads"], box, 1.0,
                                                        1e-3, seed)
    elif case["shells"]:
        out["template"] = I.icosphere(case["subdivisions"], case["radius"])
        cen = I.shell_centres(case["shells"], case["radius"], box, case["wall"], 4.0, 3.0, seed)
        out["pos"] = np.vstack([c + out["template"] for c in cen])
    elif case["particles"]:
        g = np.random.default_rng(seed)
        out["pos"] = g.uniform(0.0, 1.0, (case["particles"], 3)) * np.array(box, dtype=float)
        if case["wall"]:  # stay inside the channel
            out["pos"][:, 1] = 1.0 + (case["ny"] - 3.0) * out["pos"][:, 1] / case["ny"]
        out["vel"] = g.normal(0.0, 1e-3, (case["particles"], 3))
    return out


def _params(case):
    massive = case["coupling"] in ("fc", "ebf")
    return dict(tau=case["tau"], body_force=(0.0, 0.0, case["force"]),
                collision=COLLISION[case["collision"]], coupling=COUPLING[case["coupling"]],
                gamma=case["gamma"] if massive else 0.0, kernel=case["kernel"],
                storage=STORAGE[case["storage"]],
                f16_scale_log2=F16_SCALE if STORED_BYTES[case["storage"]] == 2 else 0,
                mts_substeps=case["substeps"], mts_inside=int(case["inside"]), kT=case["kT"],
                seed=7 if case["kT"] else 0, mrt_rates=MRT_RATES,
                deterministic=int(case["deterministic"]))


def _requests(case, seed):
    """The case's mix of periodic boxes, all there at the start: side and particle count
    log-uniform, tau and body force uniform.  The mix belongs to the case, the particles to the
    seed."""
    if case["kind"] == "ensemble":
        more = dict(fext_max=1e-6)
    else:
        more = dict(steps_range=(case["low_steps"], case["high_steps"]))
    reqs = I.serving_requests(case["boxes"], 1.0, case["mix"], np_range=(10, case["most_particles"]),
                              side_range=(case["low"], case["high"]), **more)
    g = np.random.default_rng(seed)
    for r in reqs:
        r.arrival, r.seed = 0.0, int(g.integers(0, 2**31 - 1))
    return reqs


def prepare(case, seed):
    if case["kind"] == "serving":
        reqs = _requests(case, seed)
        return dict(case=case, requests=reqs, keep={r.rid for r in reqs[::4]})
    if case["kind"] == "ensemble":
        storage = STORAGE[case["storage"]]
        reqs = _requests(case, seed)
        params = [S.request_params(r, storage, comoving=1) for r in reqs]
        pool = sum(L.ensemble_footprint(r.side, r.side, r.side, max_particles=r.nparticles, **p)
                   for r, p in zip(reqs, params)) + (64 << 20)
        ens = L.Ensemble(pool, len(reqs), storage=storage)
        slots = []
        for r, p in zip(reqs, params):
            slot, lat = ens.admit(r.side, r.side, r.side, 1 << 40, max_particles=r.nparticles, **p)
            lat.lb_init_fluid()
            pos, vel, mass = S.request_particles(r)
            lat.lb_set_particles(torch.from_numpy(pos), torch.from_numpy(vel),
                                 torch.from_numpy(mass))
            slots.append((slot, lat))
        return dict(case=case, ens=ens, slots=slots)
    p = _particles(case, seed)
    n = 0 if p["pos"] is None else len(p["pos"])
    lat = L.Lattice(case["nx"], case["ny"], case["nz"], wall_y=int(case["wall"]), max_particles=n,
                    max_bonds=0 if p["bonds"] is None else len(p["bonds"]),
                    max_shells=case["shells"],
                    max_shell_size=0 if p["template"] is None else len(p["template"]),
                    **_params(case))
    lat.lb_init_fluid(None, _flow(case, seed))
    if n:
        lat.lb_set_particles(torch.from_numpy(p["pos"]),
                             None if p["vel"] is None else torch.from_numpy(p["vel"]),
                             None if p["vel"] is None else torch.ones(n, dtype=torch.float64))
    if p["bonds"] is not None:
        lat.lb_set_bonds(p["bonds"], 30.0, 1.0)
    if p["template"] is not None:
        lat.lb_set_shells(case["shells"], p["template"], 0.05)
    return dict(case=case, lat=lat, n=n)


# --------------------------------------------------------------------- pass
def run(state):
    case = state["case"]
    if case["kind"] == "serving":
        results, fields = S.serve_batched(state["requests"], 6 << 30, max_slots=16,
                                          keep=state["keep"])
        results = sorted(results, key=lambda r: r.rid)
        return dict(momentum=np.stack([r.totals[1:7] for r in results]).astype(np.float32),
                    fields=[fields[k].astype(np.float32) for k in sorted(fields)])
    if case["kind"] == "ensemble":
        ens = state["ens"]
        ens.step(case["steps"])
        frames = []
        for slot, lat in state["slots"]:
            ens.query(slot)  # waits, and brings the slot's handle up to date
            frames.append(lat.lb_moments()[1].float())
        return frames
    lat = state["lat"]
    lat.lb_step(case["steps"])
    single = (lambda t: t) if case["storage"] == "f64" else (lambda t: t.float())
    rho, u = lat.lb_moments()
    out = dict(rho=single(rho), u=single(u))
    if case["frame"] == "all":
        out["populations"] = single(lat.lb_populations())
        out["stress"] = single(lat.lb_stress())
    if state["n"]:
        pos, vel = lat.lb_get_particles()
        out["pos"] = single(pos)
        if case["coupling"] != "ib":
            out["vel"] = single(vel)
    return out


# --------------------------------------------------------------------- work
def _box_work(sites, stored, steps, particles, nodes, couplings, frame_bytes):
    """Populations read and written once per step, and once more (19 values) at the stencil nodes
    of the particles; per particle and coupling evaluation its state and the nodes' forces."""
    per_step = particles * nodes * 19.0 * stored + couplings * particles * (48.0 + nodes * 24.0)
    return dict(bytes=steps * (38.0 * stored * sites + per_step) + frame_bytes,
                flops=steps * (FLOPS_PER_SITE * sites + couplings * particles * nodes * 60.0))


def work(case):
    if case["kind"] == "box":
        sites, stored = case["nx"] * case["ny"] * case["nz"], STORED_BYTES[case["storage"]]
        n = max(case["particles"], case["chains"] * case["beads"])
        if case["shells"]:
            n = case["shells"] * (10 * 4 ** case["subdivisions"] + 2)
        couplings = 2 * case["substeps"] if case["inside"] else 2
        width = 8 if case["storage"] == "f64" else 4
        frame = sites * (19.0 * stored + 4.0 * width) + 48.0 * n
        if case["frame"] == "all":
            frame += sites * 25.0 * width
        return _box_work(sites, stored, case["steps"], n, case["kernel"] ** 3, couplings, frame)
    if case["kind"] == "ensemble":
        reqs = _requests(case, 1)
        steps, stored = [case["steps"]] * len(reqs), STORED_BYTES[case["storage"]]
    else:
        reqs = _requests(case, 1)
        steps, stored = [r.steps for r in reqs], 2
    total = dict(bytes=0.0, flops=0.0)
    for r, n in zip(reqs, steps):
        w = _box_work(r.side ** 3, stored, n, r.nparticles, 8, 2, r.side ** 3 * (19.0 * stored + 12.0))
        total = {k: total[k] + w[k] for k in total}
    return total


# -------------------------------------------------------------------- exact
_C = np.array([(0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1),
               (1, 1, 0), (-1, -1, 0), (1, -1, 0), (-1, 1, 0), (1, 0, 1), (-1, 0, -1),
               (1, 0, -1), (-1, 0, 1), (0, 1, 1), (0, -1, -1), (0, 1, -1), (0, -1, 1)])
_OPP = [0, 2, 1, 4, 3, 6, 5, 8, 7, 10, 9, 12, 11, 14, 13, 16, 15, 18, 17]
_W = np.array([1 / 3 if not c.any() else (1 / 18 if abs(c).sum() == 1 else 1 / 36) for c in _C])
# deviate of a site that belongs to each velocity: the velocity's rank in lexical order of (x, y, z)
_RANK = np.argsort(np.argsort(9 * _C[:, 0] + 3 * _C[:, 1] + _C[:, 2]))


def _basis():
    """Moment rows of D3Q19, orthogonal under the weights: density, momentum, bulk, five shear,
    three vector ghosts, three pseudo-vector ghosts, scalar ghost, two tensor ghosts."""
    x, y, z = _C.T.astype(float)
    c2 = x * x + y * y + z * z
    E = np.stack([np.ones(19), x, y, z, c2 - 1, 3 * x * x - c2, y * y - z * z, x * y, y * z, z * x,
                  x * (3 * c2 - 5), y * (3 * c2 - 5), z * (3 * c2 - 5), x * (y * y - z * z),
                  y * (z * z - x * x), z * (x * x - y * y), 3 * c2 * c2 - 6 * c2 + 1,
                  (2 * c2 - 3) * (3 * x * x - c2), (2 * c2 - 3) * (y * y - z * z)])
    return E, (E * E) @ _W


def _rates(case):
    lam = np.full(19, 1.0 / case["tau"])
    odd = np.r_[1:4, 10:16]
    if case["collision"] == "trt":
        lam[odd] = 1.0 / (0.5 + MAGIC / (case["tau"] - 0.5))
    if case["collision"] == "mrt":
        lam[4], lam[10:13], lam[13:16], lam[16], lam[17:19] = MRT_RATES
    return lam


def _philox(c, key):
    """Philox4x32-10 of int64 tensors holding 32-bit words."""
    m = 0xFFFFFFFF

    def mul(a, x):
        low, high = a * (x & 0xFFFF), a * (x >> 16)
        return (high + (low >> 16)) >> 16, (low + ((high & 0xFFFF) << 16)) & m

    k0, k1 = key & m, key >> 32
    for _ in range(10):
        h0, l0 = mul(0xD2511F53, c[0])
        h1, l1 = mul(0xCD9E8D57, c[2])
        c = [(h1 ^ c[1]) ^ k0, l1, (h0 ^ c[3]) ^ k1, l0]
        k0, k1 = (k0 + 0x9E3779B9) & m, (k1 + 0xBB67AE85) & m
    return c


def _normals(c, key):
    u = [((x >> 9).double() + 0.5) / 8388608.0 for x in _philox(c, key)]
    out = []
    for a, b in ((u[0], u[1]), (u[2], u[3])):
        r = torch.sqrt(-2.0 * torch.log(a))
        out += [r * torch.cos(2.0 * math.pi * b), r * torch.sin(2.0 * math.pi * b)]
    return out


def _phi(K, r):
    a = r.abs()
    if K == 2:
        return torch.clamp(1 - a, min=0)
    if K == 3:
        inner = (1 + torch.sqrt(torch.clamp(1 - 3 * a * a, min=0))) / 3
        outer = (5 - 3 * a - torch.sqrt(torch.clamp(-2 + 6 * a - 3 * a * a, min=0))) / 6
        return torch.where(a <= 0.5, inner, torch.where(a <= 1.5, outer, torch.zeros_like(a)))
    inner = (3 - 2 * a + torch.sqrt(torch.clamp(1 + 4 * a - 4 * a * a, min=0))) / 8
    outer = (5 - 2 * a - torch.sqrt(torch.clamp(-7 + 12 * a - 4 * a * a, min=0))) / 8
    return torch.where(a <= 1, inner, torch.where(a <= 2, outer, torch.zeros_like(a)))


class _Exact:
    """One box in 64 bits: populations [19, N] as deviations from the weights (rho0 = 1)."""

    def __init__(self, case, p, u=None, fext=None):
        self.case, self.t = case, 0
        self.dims = (case["nz"], case["ny"], case["nx"])
        self.N = case["nx"] * case["ny"] * case["nz"]
        tensor = lambda v: torch.as_tensor(np.asarray(v), dtype=torch.float64, device="cuda")  # noqa: E731
        self.c, self.w = tensor(_C), tensor(_W)[:, None]
        E, b = _basis()
        self.lam = _rates(case)
        self.relax = tensor(np.eye(19) - _W[:, None] * (E.T * (np.r_[np.zeros(4), self.lam[4:]] / b)) @ E)
        mu = 3.0 * case["kT"]
        amp = np.sqrt(mu * self.lam * (2.0 - self.lam)) / b
        amp[:4] = 0.0
        self.noise = tensor(_W[:, None] * (E.T * amp) @ (E * np.sqrt(_W)))
        self.fext = tensor(fext if fext is not None else (0.0, 0.0, case["force"]))
        v = torch.zeros((3, self.N), dtype=torch.float64, device="cuda") if u is None else u.reshape(3, -1)
        zero = torch.zeros(self.N, dtype=torch.float64, device="cuda")
        self.f = self.feq(zero, zero + 1.0, v)
        self.box = tensor([case["nx"], case["ny"], case["nz"]])
        self.pos = None if p["pos"] is None else self.wrap(tensor(p["pos"]))
        self.vel = None if p["vel"] is None else tensor(p["vel"])
        self.bonds = None if p["bonds"] is None else torch.as_tensor(p["bonds"].astype(np.int64), device="cuda")
        self.template = None if p["template"] is None else tensor(p["template"])

    def wrap(self, x):
        y = x - self.box * torch.floor(x / self.box)
        if self.case["wall"]:
            y[:, 1] = x[:, 1]
        return y

    def nearest(self, d):
        m = d - self.box * torch.floor(d / self.box + 0.5)
        if self.case["wall"]:
            m[..., 1] = d[..., 1]
        return m

    def feq(self, d, rho, u):
        cu = self.c @ u
        return self.w * (d + rho * (3.0 * cu + 4.5 * cu * cu - 1.5 * (u * u).sum(0)))

    def moments(self):
        d = self.f.sum(0)
        return d, 1.0 + d, (self.c.T @ self.f) / (1.0 + d)

    def force(self, Fc, dt):
        """f <- f + dt G(F, u + dt F / 2 rho), which is the difference of two equilibria."""
        d, rho, u = self.moments()
        F = self.fext[:, None] + (0.0 if Fc is None else Fc)
        self.f += self.feq(d, rho, u + dt * F / rho) - self.feq(d, rho, u)

    def collide_stream(self):
        d, rho, u = self.moments()
        eq = self.feq(d, rho, u)
        f = eq + self.relax @ (self.f - eq)
        if self.case["kT"] > 0:
            site = torch.arange(self.N, device="cuda")
            g = []
            for k in range(5):
                g += _normals([site, torch.full_like(site, self.t), torch.full_like(site, k),
                               torch.zeros_like(site)], 7)
            f += torch.sqrt(rho) * (self.noise @ torch.stack([g[k] for k in _RANK]))
        f = f.reshape((19,) + self.dims)
        new = torch.empty_like(f)
        for i, (cx, cy, cz) in enumerate(_C):
            new[i] = torch.roll(f[i], (int(cz), int(cy), int(cx)), (0, 1, 2))
            if self.case["wall"] and cy:
                y = 0 if cy > 0 else self.dims[1] - 1
                new[i][:, y] = f[_OPP[i]][:, y]
        self.f = new.reshape(19, -1)
        self.t += 1

    def stencil(self, X):
        """Sites [n, K^3] and weights (zero beyond a wall)."""
        K = self.case["kernel"]
        first = (torch.floor(X + 0.5) if K == 3 else torch.floor(X)) - (0 if K == 2 else 1)
        j = first[:, :, None] + torch.arange(K, dtype=torch.float64, device="cuda")
        w = _phi(K, j - X[:, :, None])
        n = (self.case["nx"], self.case["ny"], self.case["nz"])
        if self.case["wall"]:
            w[:, 1] = torch.where((j[:, 1] < 0) | (j[:, 1] >= n[1]), torch.zeros_like(w[:, 1]), w[:, 1])
        jx, jy, jz = (torch.remainder(j[:, a], n[a]).long() for a in range(3))
        site = (jz[:, :, None, None] * n[1] + jy[:, None, :, None]) * n[0] + jx[:, None, None, :]
        W = w[:, 2, :, None, None] * w[:, 1, None, :, None] * w[:, 0, None, None, :]
        return site.reshape(len(X), -1), W.reshape(len(X), -1)

    def interpolate(self, X):
        site, W = self.stencil(X)
        f = self.f[:, site.reshape(-1)]
        rho = 1.0 + f.sum(0)
        u = (self.c.T @ f) / rho
        return (W * rho.reshape(W.shape)).sum(1), (W * u.reshape((3,) + W.shape)).sum(2).T

    def spread(self, X, F):
        site, W = self.stencil(X)
        out = torch.zeros((3, self.N), dtype=torch.float64, device="cuda")
        for a in range(3):
            out[a].index_add_(0, site.reshape(-1), (W * F[:, a, None]).reshape(-1))
        return out

    def intrinsic(self, X):
        F = torch.zeros_like(X)
        if self.bonds is not None:
            i, j = self.bonds[:, 0], self.bonds[:, 1]
            d = self.nearest(X[j] - X[i])
            length = d.norm(dim=1, keepdim=True)
            s = 30.0 * (length - 1.0) / length * d
            F.index_add_(0, i, s)
            F.index_add_(0, j, -s)
        if self.template is not None:
            Y = X.reshape(self.case["shells"], -1, 3)
            Y = Y[:, :1] + self.nearest(Y - Y[:, :1])
            Y = Y - Y.mean(1, keepdim=True)
            A = self.template.T @ Y  # [shell, 3, 3], template x marker
            U, _, Vh = torch.linalg.svd(A)
            D = torch.ones(len(A), 3, dtype=torch.float64, device="cuda")
            D[:, 2] = torch.linalg.det(U @ Vh)
            R = Vh.transpose(1, 2) @ (D[:, :, None] * U.transpose(1, 2))
            F += (-0.05 * (Y - (R @ self.template.T).transpose(1, 2))).reshape(-1, 3)
        return F

    def couple(self, Fi, hh, k):
        """Coupling over a time hh (masses 1): kicks the particles, returns the lattice force."""
        g = self.case["gamma"]
        rp, up = self.interpolate(self.pos)
        al, be = g * hh, (g * hh / rp)[:, None]
        if self.case["coupling"] == "fc":
            top = -(g * (self.vel - up) + 0.5 * al * Fi - 0.5 * be * self.fext)
            if self.case["kT"] > 0:
                p = torch.arange(len(self.pos), device="cuda")
                z = _normals([p, torch.full_like(p, self.t), torch.full_like(p, 65536 + k),
                              torch.zeros_like(p)], 7)
                top = top + math.sqrt(2.0 * self.case["kT"] * g / hh) * torch.stack(z[:3], 1)
            Fh = top / (1.0 + 0.5 * al + 0.5 * be)
            self.vel = self.vel + hh * (Fh + Fi)
        else:
            d = self.vel - up
            Fh = -(g * d + al * Fi) / (al + be)
            self.vel = self.vel - al / (al + be) * d + hh * be / (al + be) * Fi
        return self.spread(self.pos, -Fh)

    def drift(self, dt):
        self.pos = self.wrap(self.pos + dt * self.vel)

    def verlet(self, n, dt):
        for _ in range(n):
            self.drift(0.5 * dt)
            self.vel = self.vel + dt * self.intrinsic(self.pos)
            self.drift(0.5 * dt)

    def step(self):
        n, before = self.case["substeps"], self.t
        if self.pos is None:
            self.force(None, 0.5)
            self.collide_stream()
            self.force(None, 0.5)
        elif self.case["coupling"] == "ib":
            Xt = self.wrap(self.pos + 0.5 * self.interpolate(self.pos)[1])
            self.pos = self.wrap(self.pos + 0.5 * self.interpolate(Xt)[1])
            Fc = self.spread(Xt, self.intrinsic(Xt))
            self.force(Fc, 0.5)
            self.collide_stream()
            self.force(Fc, 0.5)
            self.pos = self.wrap(self.pos + 0.5 * self.interpolate(Xt)[1])
        elif n and self.case["inside"]:
            dt = 0.5 / n
            for side in (0, 1):
                for k in range(n):
                    self.drift(0.5 * dt)
                    self.force(self.couple(self.intrinsic(self.pos), dt, side * n + k), dt)
                    self.drift(0.5 * dt)
                if side == 0:
                    self.collide_stream()
                    self.t = before  # the step's random numbers carry its index
        elif n:
            none = torch.zeros_like(self.pos)
            self.force(self.couple(none, 0.5, 0), 0.5)
            self.verlet(n, 0.5 / n)
            self.collide_stream()
            self.t = before
            self.verlet(n, 0.5 / n)
            self.force(self.couple(none, 0.5, 1), 0.5)
        else:
            self.drift(0.5)
            Fi = self.intrinsic(self.pos)
            self.force(self.couple(Fi, 0.5, 0), 0.5)
            self.collide_stream()
            self.t = before
            self.force(self.couple(Fi, 0.5, 1), 0.5)
            self.drift(0.5)
        self.t = before + 1

    def stress(self):
        d, rho, u = self.moments()
        n = self.f - self.feq(d, rho, u)
        cc = torch.stack([self.c[:, a] * self.c[:, b] for a, b in ((0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2))])
        s = cc @ n
        trace = s[:3].sum(0) / 3.0
        shear, bulk = 1.0 - 0.5 * self.lam[5], 1.0 - 0.5 * self.lam[4]
        s *= shear
        s[:3] += (bulk - shear) * trace
        return s.reshape((6,) + self.dims)


def _request_box(r):
    case = _box(nx=r.side, ny=r.side, nz=r.side, tau=r.tau, particles=r.nparticles)
    pos, vel, _ = S.request_particles(r)
    return _Exact(case, dict(pos=pos, vel=vel, bonds=None, template=None), fext=(r.fext, 0.0, 0.0))


def exact(case, seed):
    if case["kind"] == "ensemble":
        frames = []
        for r in _requests(case, seed):
            e = _request_box(r)
            for _ in range(case["steps"]):
                e.step()
            frames.append(e.moments()[2].reshape((3,) + e.dims))
        return frames
    if case["kind"] == "serving":
        reqs = _requests(case, seed)
        if sum(r.side ** 3 * r.steps for r in reqs) > 4e9:
            return None
        momentum, fields = [], []
        for k, r in enumerate(reqs):
            e = _request_box(r)
            for _ in range(r.steps):
                e.step()
            d, rho, u = e.moments()
            momentum.append(torch.cat([(rho * u).sum(1), e.vel.sum(0)]))
            if k % 4 == 0:
                fields.append(u.reshape((3,) + e.dims).cpu().numpy())
        return dict(momentum=torch.stack(momentum).cpu().numpy(), fields=fields)
    e = _Exact(case, _particles(case, seed), _flow(case, seed))
    for _ in range(case["steps"]):
        e.step()
    d, rho, u = e.moments()
    out = dict(rho=rho.reshape(e.dims), u=u.reshape((3,) + e.dims))
    if case["frame"] == "all":
        out["populations"] = e.f.reshape((19,) + e.dims)
        out["stress"] = e.stress()
    if e.pos is not None:
        out["pos"] = e.pos
        if case["coupling"] != "ib":
            out["vel"] = e.vel
    return out
