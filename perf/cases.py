"""The work that users of this solver have it do, as cases that can be timed and checked.

A pass advances a simulation by ``steps`` time steps through ``lbib.Sim`` or ``lbib.Batch`` and reads the fields
(density, velocity) and the capsules' state back on the device, or takes one gradient.  A simulation in FP32 keeps what
it reads in FP32.

A pass of the Dynamic coupling, or with the contact force, starts again from a state saved on the device: both run a
window of a few hundred steps from a given state (the Dynamic scheme leaves the finite range after that), as in a
parameter study that restarts from a checkpoint.  The other passes go on from where the last one ended.

``exact`` computes the same numbers with plain torch operations in 64 bits: the D2Q9 BGK step with Guo forcing, the
Zou-He boundaries, the MLS interpolation and spreading, the membrane, contact and hydrodynamic forces, and the
Kinematic and Dynamic node updates; its gradients come from torch's autograd.
"""
import math

import numpy as np
import torch

TAU, U_MAX = 0.8, 0.02
NU = (TAU - 0.5) / 3.0
WARM = 2  # steps before the saved state


def listed():
    return [
        # one step at a time of the 64 x 64 FP64 shear capsule, the reference configuration: launches and latency only
        dict(name="shear64_fp64_1step", kind="shear", nx=64, ny=64, caps=1, nodes=64, size=8.0, real_bytes=8,
             mode="kinematic", steps=1),
        # a capsule migrating across a Couette flow, small lattice, long runs: the launch of the capsule kernel counts
        dict(name="couette256x101_kin", kind="shear", nx=256, ny=101, caps=1, nodes=100, size=12.5, real_bytes=4,
             mode="kinematic", steps=100),
        # one biconcave capsule in a channel, the configuration of the single-capsule studies
        dict(name="channel1024x256_dyn", kind="channel", nx=1024, ny=256, caps=1, nodes=128, size=20.0, real_bytes=4,
             mode="dynamic", steps=100),
        # many inertial capsules in a mid-size channel
        dict(name="channel2048x512_dyn_32", kind="channel", nx=2048, ny=512, caps=32, nodes=128, size=9.0,
             real_bytes=4, mode="dynamic", steps=100),
        # the benchmark's headline step
        dict(name="channel4096_dyn_32", kind="channel", nx=4096, ny=4096, caps=32, nodes=128, size=9.0, real_bytes=4,
             mode="dynamic", steps=50),
        # the fluid alone, in both precisions, the FP64 one on odd sizes
        dict(name="grid4096_fp32", kind="channel", nx=4096, ny=4096, caps=0, nodes=0, size=0.0, real_bytes=4,
             mode="kinematic", steps=40),
        dict(name="grid1777x1003_fp64", kind="channel", nx=1777, ny=1003, caps=0, nodes=0, size=0.0, real_bytes=8,
             mode="kinematic", steps=41),
        # a dense suspension: every capsule touches its neighbours (contact force, four by four block)
        dict(name="dense130x81_kin_16", kind="dense", nx=130, ny=81, caps=16, nodes=96, size=15.0, real_bytes=4,
             mode="kinematic", steps=100),
        # capsules and rigid discs in contact in an open channel (velocity inlet, pressure outlet)
        dict(name="open1536x256_dyn_16", kind="open", nx=1536, ny=256, caps=16, nodes=96, size=15.0, real_bytes=4,
             mode="dynamic", steps=60),
        # an ensemble of small channels of all sizes, stepped as one batch
        dict(name="ensemble256_kin", kind="ensemble", nx=512, ny=128, caps=2, nodes=128, size=9.0, real_bytes=4,
             mode="kinematic", steps=200, lattices=256),
        # gradients of the final deformation: whole trajectory in memory, and with checkpoints
        dict(name="gradient512x128_dyn", kind="gradient", nx=512, ny=128, caps=1, nodes=96, size=10.0, real_bytes=4,
             mode="dynamic", steps=200, every=0),
        dict(name="gradient512x128_kin_ckpt", kind="gradient", nx=512, ny=128, caps=1, nodes=96, size=10.0,
             real_bytes=4, mode="kinematic", steps=280, every=70),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["shear", "channel", "channel", "channel", "grid", "grid", "dense", "open", "ensemble",
                       "gradient"])
    mode = rng.choice(["dynamic", "kinematic"])
    rb = rng.choice([4, 4, 8])
    if kind == "shear":
        ny = _log(rng, 64, 256)
        size = rng.uniform(0.08, 0.13) * ny
        return dict(kind=kind, nx=_log(rng, 64, 512), ny=ny, caps=1, nodes=_nodes(rng, size), size=size,
                    real_bytes=rb, mode="kinematic", steps=_log(rng, 1, 100))
    if kind == "channel":
        nx, ny = _log(rng, 128, 4096), _log(rng, 64, 2048)
        size = rng.uniform(6.0, min(20.0, ny / 6.0))
        room = int(nx // (2.0 * size + 16.0)) * int((ny - 12) // (2.0 * size + 10.0))
        caps = max(1, min(room, _log(rng, 1, 64)))
        return dict(kind=kind, nx=nx, ny=ny, caps=caps, nodes=_nodes(rng, size), size=size, real_bytes=rb, mode=mode,
                    steps=rng.randint(10, 50))
    if kind == "grid":
        return dict(kind="channel", nx=_log(rng, 32, 4096), ny=_log(rng, 32, 2048), caps=0, nodes=0, size=0.0,
                    real_bytes=rb, mode="kinematic", steps=rng.randint(1, 40))
    if kind == "dense":
        size = rng.uniform(12.0, 18.0)
        nx = int(math.ceil(4.0 * (2.0 * size + 2.5)))
        ny = int(math.ceil(4.0 * (size + 2.5) + 11.0))
        return dict(kind=kind, nx=nx, ny=ny, caps=16, nodes=_nodes(rng, size), size=size, real_bytes=rb,
                    mode="kinematic", steps=rng.randint(10, 100))
    if kind == "open":
        return dict(kind=kind, nx=_log(rng, 384, 2048), ny=rng.randint(120, 320), caps=16, nodes=96,
                    size=rng.uniform(12.0, 15.0), real_bytes=rb, mode="dynamic", steps=rng.randint(10, 60))
    if kind == "ensemble":
        return dict(kind=kind, nx=rng.randint(200, 512), ny=rng.randint(80, 128), caps=2, nodes=rng.randint(80, 128),
                    size=rng.uniform(7.0, 9.0), real_bytes=4, mode=rng.choice(["kinematic"]),
                    steps=rng.randint(50, 200), lattices=_log(rng, 4, 256))
    size = rng.uniform(7.0, 11.0)
    return dict(kind="gradient", nx=_log(rng, 96, 512), ny=rng.randint(64, 128), caps=1, nodes=_nodes(rng, size),
                size=size, real_bytes=rb, mode=mode, steps=rng.randint(40, 200), every=rng.choice([0, 0, 30, 70]))


def _nodes(rng, size):
    """Node count that keeps the element length of a capsule of half-length `size` between 0.6 and 0.9."""
    return int(2.0 * math.pi * size / rng.uniform(0.6, 0.9)) + 1


# ------------------------------------------------------------------ inputs
def _circle(cx, cy, r, n):
    a = 2.0 * math.pi * (np.arange(n) + 0.5) / n
    return np.stack([cx + r * np.cos(a), cy + r * np.sin(a)], 1)


def _biconcave(cx, cy, half, n, angle):
    """Biconcave outline with n nodes at equal arc lengths, counter-clockwise."""
    q = -0.5 * math.pi + 2.0 * math.pi * np.arange(8000) / 8000
    s = np.sin(q)
    c = np.stack([half * s, 0.5 * half * (0.207 + 2.003 * s ** 2 - 1.123 * s ** 4) * np.cos(q)], 1)[::-1]
    c = np.vstack([c, c[:1]])
    arc = np.concatenate([[0.0], np.cumsum(np.hypot(*np.diff(c, axis=0).T))])
    at = np.arange(n) * (arc[-1] / n)
    p = np.stack([np.interp(at, arc, c[:, 0]), np.interp(at, arc, c[:, 1])], 1)
    ca, sa = math.cos(angle), math.sin(angle)
    return p @ np.array([[ca, sa], [-sa, ca]]) + np.array([cx, cy])


def _area(p):
    x, y = p[:, 0], p[:, 1]
    return 0.5 * float(np.sum(x * np.roll(y, -1) - np.roll(x, -1) * y))


def _membrane(p, ks, ratio=1.0, kb=0.0):
    p = np.ascontiguousarray(p)
    return dict(nodes=p, ks=float(ks), kb=float(kb), ka=1.0, mass=ratio * _area(p), density_ratio=ratio)


def _disc(cx, cy, r, n):
    p = np.ascontiguousarray(_circle(cx, cy, r, n))
    x, y = (p - p.mean(0)).T
    xn, yn = np.roll(x, -1), np.roll(y, -1)
    cr = x * yn - xn * y
    j = ((x * x + x * xn + xn * xn + y * y + y * yn + yn * yn) * cr).sum() / 12.0
    return dict(nodes=p, rigid=True, ks=0.0, kb=0.0, ka=0.0, mass=_area(p), inertia=float(j), density_ratio=1.0)


def _lattice(case, nx, ny, tau=TAU, **kw):
    cfg = dict(name=case["kind"], nx=nx, ny=ny, tau=tau, real_bytes=case["real_bytes"], mode=case["mode"], steps=0,
               periodic_y=0, u_bottom=0.0, u_top=0.0, body_force_x=0.0, init_profile=0, init_u=(0.0, 0.0), capsules=[])
    cfg.update(kw)
    return cfg


def _channel(case, nx, ny, u, tau=TAU):
    """Periodic channel driven by the body force for the peak speed u, started from the parabola."""
    return _lattice(case, nx, ny, tau, body_force_x=8.0 * (tau - 0.5) / 3.0 * u / (ny - 1) ** 2, init_profile=2)


def _capsule(rng, cx, cy, size, n, u, nu=NU):
    """Circular or biconcave capsule of half-length `size`, Ca between 1e-2 and 1e-1, density ratio 1 to 2."""
    ks = nu * u / 10.0 ** rng.uniform(-2.0, -1.0)
    ratio = rng.uniform(1.0, 2.0)
    if rng.uniform() < 0.5:
        return _membrane(_biconcave(cx, cy, size, n, rng.uniform(0.0, 2.0 * math.pi)), ks, ratio)
    return _membrane(_circle(cx, cy, size, n), ks, ratio)


def _config(case, seed):
    """Workload dictionary of a case (a list of them for an ensemble)."""
    rng = np.random.default_rng(seed)
    kind, nx, ny, n, size = case["kind"], case["nx"], case["ny"], case["nodes"], case["size"]
    u = U_MAX * rng.uniform(0.9, 1.1)
    if kind == "shear":
        cfg = _lattice(case, nx, ny, u_bottom=-0.5 * u, u_top=0.5 * u, init_profile=1)
        ks = NU * u / 10.0 ** rng.uniform(-2.0, -1.5)
        c = (nx * rng.uniform(0.4, 0.6), (ny - 1) * rng.uniform(0.45, 0.55))
        cfg["capsules"] = [_membrane(_circle(*c, size, n), ks, kb=0.05 * ks)]
    elif kind == "channel":
        cfg = _channel(case, nx, ny, u)
        if case["caps"] == 1:
            y = rng.uniform(size + 5.0, ny - 1 - size - 5.0)
            cfg["capsules"] = [_capsule(rng, nx * rng.uniform(0.2, 0.8), y, size, n, u)]
        else:  # on a grid of places with room for every orientation, moved about at random within it
            cols = max(1, int(nx // (2.0 * size + 16.0)))
            rows = max(1, int((ny - 12) // (2.0 * size + 10.0)))
            at = rng.permutation(cols * rows)[:case["caps"]]
            px, py = nx / cols, (ny - 12.0) / rows
            for k in at:
                jx, jy = rng.uniform(-1, 1, 2) * np.maximum(0.0, [0.5 * px - size - 4.0, 0.5 * py - size - 3.0])
                cfg["capsules"].append(_capsule(rng, (k % cols + 0.5) * px + jx, 6.0 + (k // cols + 0.5) * py + jy,
                                                size, n, u))
    elif kind == "dense":
        cfg = _channel(case, nx, ny, u)
        ks = NU * u / 1e-2
        for k in range(case["caps"]):
            jx, jy = rng.uniform(-1.0, 1.0, 2)
            cfg["capsules"].append(_membrane(_biconcave(
                (k % 4 + 0.5) * nx / 4.0 + jx, 0.5 * (ny - 1) + (k // 4 - 1.5) * (size + 2.5) + jy, size, n,
                rng.uniform(-0.1, 0.1)), ks))
        cfg["contact_cutoff"] = 2.0
    elif kind == "open":
        cfg = _lattice(case, nx, ny, periodic_x=0, inlet_umax=u, outlet_rho=1.0, init_profile=4)
        ks = NU * u / 1e-2
        for k in range(case["caps"]):
            jx, jy = rng.uniform(-1.0, 1.0, 2)
            cx = 0.25 * nx + (k % 4) * (2.0 * size + 2.5) + jx
            cy = 0.5 * (ny - 1) + (k // 4 - 1.5) * (size + 2.5) + jy
            a = rng.uniform(-0.3, 0.3)
            cfg["capsules"].append(_disc(cx, cy, 0.5 * size, 64) if k < 2
                                   else _membrane(_biconcave(cx, cy, size, n, a), ks))
        cfg["contact_cutoff"] = 2.0
    elif kind == "ensemble":
        cfg = []
        sizes = np.random.default_rng([nx, ny, case["lattices"]])  # the same lattices for every seed
        for _ in range(case["lattices"]):
            lx, ly = int(sizes.integers(nx // 4, nx + 1)), int(sizes.integers(ny // 2 + 8, ny + 1))
            tau = rng.uniform(0.6, 1.2)
            c = _channel(case, lx, ly, u, tau)
            m = min(int(sizes.integers(1, case["caps"] + 1)), max(1, int(lx // (2.0 * size + 20.0))))
            for k in range(m):
                r = rng.uniform(5.0, size)
                c["capsules"].append(_capsule(rng, (k + 0.5) * lx / m + rng.uniform(-4.0, 4.0),
                                              rng.uniform(r + 4.5, ly - 1 - r - 4.5), r,
                                              int(sizes.integers(n // 2, n + 1)), u, (tau - 0.5) / 3.0))
            cfg.append(c)
    else:  # gradient
        cfg = _channel(case, nx, ny, u)
        c = (nx * rng.uniform(0.25, 0.75), (ny - 1) * rng.uniform(0.4, 0.45))
        cfg["capsules"] = [_membrane(_circle(*c, size, n), NU * u / 10.0 ** rng.uniform(-2.0, -1.5))]
    return cfg


def _disturbed(case, cfg, seed, device):
    """Populations of a capsule-free run: the channel's flow with a disturbance, [9][ny][nx]."""
    gen = torch.Generator(device=device).manual_seed(int(seed))
    f = torch.randn((9, case["ny"], case["nx"]), generator=gen, device=device, dtype=torch.float64)
    y = torch.arange(case["ny"], dtype=torch.float64, device=device)
    ux = cfg["body_force_x"] / (2.0 * NU) * y * (case["ny"] - 1 - y)
    ex = torch.tensor([e[0] for e in _E], dtype=torch.float64, device=device)
    eu = ex[:, None] * ux
    feq = _weights(device)[:, None] * (1.0 + 3.0 * eu + 4.5 * eu * eu - 1.5 * ux * ux)
    return f.mul_(0.002).add_(1.0).mul_(feq[:, :, None])


def _restarts(case):
    return case["kind"] in ("channel", "dense", "open") and (case["mode"] == "dynamic" or case["kind"] == "dense")


# ------------------------------------------------------------------ passes
class _State:
    pass


def prepare(case, seed):
    from paper_1903_03356_amd import lbib
    s = _State()
    s.case, s.cfg, s.lbib = case, _config(case, seed), lbib
    dev = torch.device("cuda")
    if case["kind"] == "gradient":
        sim = lbib.Sim(s.cfg)  # sizes the workspace that the program keeps
        s.workspace = torch.empty(sim.adjoint_bytes(case["steps"], case["every"]), dtype=torch.uint8, device=dev)
        sim.close()
        return s
    s.sim = sim = lbib.Batch(s.cfg) if case["kind"] == "ensemble" else lbib.Sim(s.cfg)
    cells = sum(3 * x * y for x, y in sim.dims)
    s.fields = torch.empty(cells, dtype=torch.float64, device=dev)
    s.nodes = torch.empty(max(1, 6 * sum(sim.nv)), dtype=torch.float64, device=dev)
    if not sim.nv:
        sim.set_pops(_disturbed(case, s.cfg, seed, dev))
    s.saved = None
    if _restarts(case):
        sim.step(WARM)
        f = torch.empty((9, case["ny"], case["nx"]), dtype=torch.float64, device=dev)
        sim.get_state(lbib.F_POPS, 0, out=f)
        caps = [sim.get_state(lbib.C_STATE, c, out=torch.empty((3, n, 2), dtype=torch.float64, device=dev))
                for c, n in enumerate(sim.nv)]
        s.saved = f, caps
    return s


def run(s):
    lbib, case = s.lbib, s.case
    if case["kind"] == "gradient":
        sim = lbib.Sim(s.cfg)
        r = sim.adjoint(case["steps"], lbib.OBJ_TAYLOR, workspace=s.workspace, checkpoint_every=case["every"])
        sim.close()
        kept = np.float32 if case["real_bytes"] == 4 else np.float64
        return {"J": kept(r["J"]), "dJ_dg": kept(r["dJ_dg"]), "dJ_dks": r["dJ_dks"][0].astype(kept)}
    sim = s.sim
    if s.saved is not None:
        sim.set_state(lbib.F_POPS, s.saved[0])
        for c, x in enumerate(s.saved[1]):
            sim.set_state(lbib.C_STATE, x, c)
    sim.step(case["steps"])
    at = 0
    fields = []
    for i, (x, y) in enumerate(sim.dims):
        sim.get_state(lbib.F_MOMENTS, i, out=s.fields[at:at + 3 * x * y])
        fields.append((at, x * y))
        at += 3 * x * y
    at = 0
    for c, n in enumerate(sim.nv):
        sim.get_state(lbib.C_STATE, c, out=s.nodes[at:at + 6 * n])
        at += 6 * n
    kept = torch.float32 if case["real_bytes"] == 4 else torch.float64
    f = s.fields.to(kept)
    out = {"fields": f} if len(fields) > 1 else {"rho": f[:fields[0][1]], "u": f[fields[0][1]:]}
    if sim.nv:
        out["nodes"] = s.nodes.to(kept)
    return out


def work(case):
    """State read once and written once, results written once; about 200 operations a cell and step."""
    rb, steps = case["real_bytes"], case["steps"]
    cells = case["nx"] * case["ny"]
    if case["kind"] == "ensemble":  # mean sizes of the drawn lattices
        cells = int(case["lattices"] * (0.625 * case["nx"]) * (0.75 * case["ny"] + 4))
    nodes = case["caps"] * case["nodes"] * case.get("lattices", 1)
    back = 4 if case["kind"] == "gradient" else 1  # the reverse step: about three times a forward one
    state = 2 * (9 * rb * cells + 8 * rb * nodes)
    out = 8 * nodes if case["kind"] == "gradient" else 3 * rb * cells + 6 * rb * nodes
    return {"bytes": state + out, "flops": back * steps * (200.0 * cells + 3000.0 * nodes)}


# ------------------------------------------------------------------- exact
_E = [(0, 0), (1, 0), (0, 1), (-1, 0), (0, -1), (1, 1), (-1, 1), (-1, -1), (1, -1)]


def _weights(device):
    return torch.tensor([4 / 9] + [1 / 9] * 4 + [1 / 36] * 4, dtype=torch.float64, device=device)


class _Exact:
    """The method in 64-bit torch operations, one lattice; f holds f^n (deviations from the weights), complete."""

    def __init__(self, cfg, device, ks=None, g=None):
        self.cfg, self.dev = cfg, device
        self.nx, self.ny, self.tau = cfg["nx"], cfg["ny"], cfg["tau"]
        self.nu = (self.tau - 0.5) / 3.0
        self.g = torch.tensor(float(cfg["body_force_x"]), dtype=torch.float64, device=device) if g is None else g
        self.open = not cfg.get("periodic_x", 1)
        t = lambda v, d=torch.float64: torch.as_tensor(np.asarray(v), dtype=d, device=device)  # noqa: E731
        y = torch.arange(self.ny, dtype=torch.float64, device=device)
        H = self.ny - 1
        prof = {0: 0.0 * y, 1: cfg["u_bottom"] + (cfg["u_top"] - cfg["u_bottom"]) * y / H,
                2: self.g / (2.0 * self.nu) * y * (H - y),
                4: 4.0 * cfg.get("inlet_umax", 0.0) * y * (H - y) / H ** 2}[cfg["init_profile"]]
        u = prof[:, None].expand(self.ny, self.nx)
        self.w = _weights(device)
        self.inlet = 4.0 * cfg.get("inlet_umax", 0.0) * y * (H - y) / H ** 2
        self.f = self.complete(self.equilibrium(torch.ones_like(u), u, torch.zeros_like(u)))
        self.F = torch.stack([self.g.expand(self.ny, self.nx), torch.zeros_like(u)])
        caps = cfg["capsules"]
        if not caps:
            return
        x = [c["nodes"] for c in caps]
        off = np.cumsum([0] + [len(p) for p in x])
        self.x = t(np.concatenate(x))
        self.x0 = self.x
        self.cap = t(np.repeat(np.arange(len(x)), [len(p) for p in x]), torch.long)
        self.nxt = t(np.concatenate([o + np.roll(np.arange(len(p)), -1) for o, p in zip(off, x)]), torch.long)
        self.prv = t(np.concatenate([o + np.roll(np.arange(len(p)), 1) for o, p in zip(off, x)]), torch.long)
        per = lambda k: t([c[k] for c in caps])[self.cap]  # noqa: E731
        self.ks = per("ks") if ks is None else ks
        self.kb, self.ka = per("kb"), per("ka")
        self.mv = t([c["mass"] / len(c["nodes"]) for c in caps])[self.cap]
        e = self.x[self.nxt] - self.x
        self.l0, self.th0 = e.norm(dim=1), self.turn(self.x)
        self.A0 = self.area(self.x)
        self.rigid = []
        for k, c in enumerate(caps):
            if c.get("rigid"):
                i = slice(int(off[k]), int(off[k + 1]))
                p = self.x[i]
                cr = p[:, 0] * p.roll(-1, 0)[:, 1] - p.roll(-1, 0)[:, 0] * p[:, 1]
                X = ((p + p.roll(-1, 0)) * cr[:, None]).sum(0) / (3.0 * cr.sum())
                self.rigid.append(dict(i=i, X=X, th=torch.zeros((), dtype=torch.float64, device=device), r0=p - X,
                                       m=c["mass"], I=c["inertia"]))
        self.d = self.uv = self.first = None

    # ---- fluid
    def equilibrium(self, rho, ux, uy):
        """Equilibrium less the weights."""
        out = []
        for i, (ex, ey) in enumerate(_E):
            eu = ex * ux + ey * uy
            out.append(self.w[i] * ((rho - 1.0) + rho * (3.0 * eu + 4.5 * eu * eu - 1.5 * (ux * ux + uy * uy))))
        return torch.stack(out)

    def moments(self):
        """rho, u with the half force of the last collision."""
        f = self.f
        rho = 1.0 + f.sum(0)
        ux = (f[1] - f[3] + f[5] - f[6] + f[8] - f[7] + 0.5 * self.F[0]) / rho
        uy = (f[2] - f[4] + f[5] + f[6] - f[7] - f[8] + 0.5 * self.F[1]) / rho
        return rho, ux, uy

    def fluid_step(self, spread):
        """Collide with F = g + spread, stream, complete the boundaries."""
        Fx, Fy = spread[0] + self.g, spread[1]
        self.F = torch.stack([Fx, Fy])
        rho, ux, uy = self.moments()
        feq = self.equilibrium(rho, ux, uy)
        om = 1.0 / self.tau
        new = []
        for i, (ex, ey) in enumerate(_E):
            eu, eF = ex * ux + ey * uy, ex * Fx + ey * Fy
            src = (1.0 - 0.5 * om) * self.w[i] * (3.0 * (eF - ux * Fx - uy * Fy) + 9.0 * eu * eF)
            new.append(torch.roll(self.f[i] - om * (self.f[i] - feq[i]) + src, (ey, ex), (0, 1)))
        self.f = self.complete(torch.stack(new))

    def complete(self, f):
        c = self.cfg
        f = f.clone()
        drho = f.sum(0) if self.open else None  # of the inner cells, for the corners
        for row, uw, top in ((0, c["u_bottom"], False), (self.ny - 1, c["u_top"], True)):
            s = f[:, row].clone()
            known = (4, 7, 8) if not top else (2, 5, 6)
            rw = 1.0 + s[0] + s[1] + s[3] + 2.0 * (s[known[0]] + s[known[1]] + s[known[2]])
            m = 0.5 * (rw * uw - 0.5 * self.g)
            h = 0.5 * (s[1] - s[3])
            if top:
                f[4, row], f[7, row], f[8, row] = s[2], s[5] + h - m, s[6] - h + m
            else:
                f[2, row], f[5, row], f[6, row] = s[4], s[7] - h + m, s[8] + h - m
        if not self.open:
            return f
        s = f[:, :, 0].clone()
        ux = self.inlet
        m = (1.0 + s[0] + s[2] + s[4] + 2.0 * (s[3] + s[6] + s[7])) / (1.0 - ux) * ux
        q = 0.5 * (s[2] - s[4])
        f[1, :, 0], f[5, :, 0], f[8, :, 0] = s[3] + 2.0 / 3.0 * m, s[7] - q + m / 6.0, s[6] + q + m / 6.0
        s = f[:, :, -1].clone()
        ro = c["outlet_rho"]
        m = 1.0 + s[0] + s[2] + s[4] + 2.0 * (s[1] + s[5] + s[8]) - ro
        q = 0.5 * (s[2] - s[4])
        f[3, :, -1], f[7, :, -1], f[6, :, -1] = s[1] - 2.0 / 3.0 * m, s[5] + q - m / 6.0, s[8] - q - m / 6.0
        inv = [0, 3, 4, 1, 2, 7, 8, 5, 6]
        for yy, yi, kn in ((0, 1, 4), (self.ny - 1, self.ny - 2, 2)):  # at rest in the corners
            for xx, xi, kx in ((0, 1, 3), (self.nx - 1, self.nx - 2, 1)):
                diag = next(i for i, e in enumerate(_E) if e == (_E[kx][0], _E[kn][1]))
                s = f[:, yy, xx].clone()
                s[inv[kx]], s[inv[kn]], s[inv[diag]] = s[kx], s[kn], s[diag]
                rest = [i for i in range(5, 9) if i not in (diag, inv[diag])]
                total = s.sum() - s[rest[0]] - s[rest[1]]
                s[rest[0]] = s[rest[1]] = 0.5 * (drho[yi, xi] - total)
                f[:, yy, xx] = s
        return f

    # ---- moving least squares
    def fit(self, p):
        """Flat indices of the 3 x 3 supports, values and slopes of the shape functions."""
        c = torch.floor(p.detach() + 0.5)
        o = torch.arange(-1, 2, device=self.dev, dtype=torch.float64)
        oy, ox = torch.meshgrid(o, o, indexing="ij")
        X = c[:, :1] + ox.reshape(1, 9) - p[:, :1]
        Y = c[:, 1:] + oy.reshape(1, 9) - p[:, 1:]
        W = torch.exp(-(X * X + Y * Y) / 0.78 ** 2)
        a = [(W * q).sum(1) for q in (torch.ones_like(X), X, Y, X * X, X * Y, Y * Y)]
        M = torch.stack([a[0], a[1], a[2], a[1], a[3], a[4], a[2], a[4], a[5]], 1)
        c00 = M[:, 4] * M[:, 8] - M[:, 5] ** 2
        c01 = M[:, 2] * M[:, 5] - M[:, 1] * M[:, 8]
        c02 = M[:, 1] * M[:, 5] - M[:, 2] * M[:, 4]
        c11 = M[:, 0] * M[:, 8] - M[:, 2] ** 2
        c12 = M[:, 1] * M[:, 2] - M[:, 0] * M[:, 5]
        c22 = M[:, 0] * M[:, 4] - M[:, 1] ** 2
        det = M[:, 0] * c00 + M[:, 1] * c01 + M[:, 2] * c02
        row = lambda i, j, k: W * (i[:, None] + j[:, None] * X + k[:, None] * Y) / det[:, None]  # noqa: E731
        ix = (c[:, :1] + ox.reshape(1, 9)).long() % self.nx
        iy = (c[:, 1:] + oy.reshape(1, 9)).long() % self.ny
        return iy * self.nx + ix, row(c00, c01, c02), row(c01, c11, c12), row(c02, c12, c22)

    def at(self, p, field):
        i, phi, _, _ = self.fit(p)
        return torch.stack([(phi * q.reshape(-1)[i]).sum(1) for q in field[1:]], 1)

    def spread(self, p, force):
        i, phi, _, _ = self.fit(p)
        out = []
        for k in range(2):
            z = torch.zeros(self.nx * self.ny, dtype=torch.float64, device=self.dev)
            out.append(z.index_add(0, i.reshape(-1), (phi * force[:, k:k + 1]).reshape(-1)).reshape(self.ny, self.nx))
        return torch.stack(out)

    def probe(self, p, field):
        i, phi, gx, gy = self.fit(p)
        r, u, v = (q.reshape(-1)[i] for q in field)
        G = [(a * b).sum(1) for a in (u, v) for b in (gx, gy)]
        return ((phi * (r - 1.0)).sum(1) / 3.0, *G)

    # ---- forces on the nodes
    def area(self, x):
        a = 0.5 * (x[:, 0] * x[self.nxt, 1] - x[self.nxt, 0] * x[:, 1])
        z = torch.zeros(int(self.cap.max()) + 1, dtype=torch.float64, device=self.dev)
        return z.index_add(0, self.cap, a)

    def turn(self, x):
        a, b = x - x[self.prv], x[self.nxt] - x
        return torch.atan2(a[:, 0] * b[:, 1] - a[:, 1] * b[:, 0], (a * b).sum(1))

    @staticmethod
    def right(v):
        return torch.stack([v[:, 1], -v[:, 0]], 1)

    def membrane(self, x):
        e = x[self.nxt] - x
        ln = e.norm(dim=1, keepdim=True)
        c = self.ks[:, None] * (ln - self.l0[:, None]) / ln * e
        a = (0.5 * self.ka * (1.0 - self.area(x) / self.A0)[self.cap] / 3.0)[:, None] * self.right(e)
        f = (c + a) + (a - c)[self.prv]
        if bool((self.kb != 0).any()):
            s = (self.kb * torch.sin(self.turn(x) - self.th0))[:, None]
            left, rgt = s * self.right(e)[self.prv] / ln[self.prv] ** 2, s * self.right(e) / ln ** 2
            f = f + rgt[self.prv] + left[self.nxt] - left - rgt
        return f

    def hydro(self, x, field):
        e = x[self.nxt] - x
        ln = e.norm(dim=1, keepdim=True)
        n, mid = self.right(e) / ln, 0.5 * (x + x[self.nxt])
        a, b = (self.probe(mid + s * n, field) for s in (1.2, -1.2))
        d = [p - q for p, q in zip(a, b)]
        f = self.traction(n, d) * ln
        return 0.5 * (f + f[self.prv])

    def traction(self, n, q):
        dp, g00, g01, g10, g11 = q
        return torch.stack([-dp * n[:, 0] + self.nu * (2.0 * g00 * n[:, 0] + (g01 + g10) * n[:, 1]),
                            -dp * n[:, 1] + self.nu * ((g01 + g10) * n[:, 0] + 2.0 * g11 * n[:, 1])], 1)

    def contact(self, x):
        cut = self.cfg.get("contact_cutoff", 0.0)
        if not cut or int(self.cap.max()) == 0:
            return torch.zeros_like(x)
        d = x[None] - x[:, None]
        dx = d[..., 0] - (0 if self.open else self.nx * torch.round(d[..., 0] / self.nx))
        r = torch.sqrt(dx * dx + d[..., 1] ** 2)
        hit = (self.cap[:, None] != self.cap[None]) & (r < cut) & (r > 0)
        mag = torch.where(hit, 1e-4 / (8.0 * math.sqrt(2.0)) * r.clamp_min(1e-9) ** -2.5, torch.zeros_like(r)).sum(1)
        e = x[self.nxt] - x
        n = self.right(e) / e.norm(dim=1, keepdim=True)
        n = n + n[self.prv]
        return -mag[:, None] * n / n.norm(dim=1, keepdim=True)

    # ---- one step
    def step(self):
        if not self.cfg["capsules"]:
            self.fluid_step(torch.zeros_like(self.F))
            return
        dyn = self.cfg["mode"] == "dynamic"
        field = self.moments()
        if self.d is None:  # start-up
            u = self.at(self.x, field)
            for q in self.rigid:
                v, r = u[q["i"]], q["r0"]
                q["u"] = q["um"] = v.mean(0)
                q["w"] = q["wm"] = (r[:, 0] * v[:, 1] - r[:, 1] * v[:, 0]).sum() / (r * r).sum()
                u = u.clone()
                u[q["i"]] = q["u"] - q["w"] * self.right(r)
            self.d = self.uv = self.first = u  # the Kinematic scheme keeps its first node velocity
        if dyn:
            e = (self.x[self.nxt] - self.x).norm(dim=1)
            cv = 0.5 * (e + e[self.prv])
            force = cv[:, None] * (self.uv - self.at(self.x, field))
        else:
            force = self.membrane(self.x) + self.contact(self.x)
        self.fluid_step(self.spread(self.x, force))
        field = self.moments()
        u = self.at(self.x, field)
        if not dyn:
            self.d = self.d / 3.0 + u * 2.0 / 3.0
            self.x = self.x + self.d
            return
        touch = self.contact(self.x)
        f = self.membrane(self.x) + self.hydro(self.x, field) + touch
        d = u + 0.5 / self.mv[:, None] * f
        uv = 1.5 * d - 0.5 * self.d
        x = self.x + d
        for q in self.rigid:
            i = q["i"]
            p, c = self.x[i], touch[i]
            e = p.roll(-1, 0) - p
            ln = e.norm(dim=1, keepdim=True)
            n, mid = self.right(e) / ln, 0.5 * (p + p.roll(-1, 0))
            t = self.traction(n, self.probe(mid + 1.2 * n, field)) * ln
            cross = lambda a, b: a[:, 0] * b[:, 1] - a[:, 1] * b[:, 0]  # noqa: E731
            M = cross(mid - q["X"], t).sum() + cross(p - q["X"], c).sum()
            u1 = 2.0 / 3.0 * (2.0 * q["u"] - 0.5 * q["um"] + (t.sum(0) + c.sum(0)) / q["m"])
            w1 = 2.0 / 3.0 * (2.0 * q["w"] - 0.5 * q["wm"] + M / q["I"])
            q["um"], q["wm"], q["u"], q["w"] = q["u"], q["w"], u1, w1
            q["X"], q["th"] = q["X"] + u1, q["th"] + w1
            cs, sn = torch.cos(q["th"]), torch.sin(q["th"])
            r = torch.stack([cs * q["r0"][:, 0] - sn * q["r0"][:, 1], sn * q["r0"][:, 0] + cs * q["r0"][:, 1]], 1)
            x[i], uv[i] = q["X"] + r, u1 - w1 * self.right(r)
            d[i] = x[i] - p
        self.x, self.d, self.uv = x, d, uv

    def taylor(self, k=0):
        """Taylor deformation of the equivalent ellipse."""
        p = self.x[self.cap == k]
        p = p - p.detach().mean(0)
        q = p.roll(-1, 0)
        cr = p[:, 0] * q[:, 1] - q[:, 0] * p[:, 1]
        A = 0.5 * cr.sum()
        c = ((p + q) * cr[:, None]).sum(0) / (6.0 * A)
        jxx, jyy = ((p * p + p * q + q * q) * cr[:, None]).sum(0) / 12.0 - A * c * c
        jxy = ((p[:, 0] * q[:, 1] + 2.0 * p[:, 0] * p[:, 1] + 2.0 * q[:, 0] * q[:, 1] + q[:, 0] * p[:, 1]) * cr
               ).sum() / 24.0 - A * c[0] * c[1]
        r = torch.sqrt(0.25 * (jxx - jyy) ** 2 + jxy ** 2)
        a, b = torch.sqrt(0.5 * (jxx + jyy) + r), torch.sqrt(0.5 * (jxx + jyy) - r)
        return (a - b) / (a + b)


def exact(case, seed):
    dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
    cfg = _config(case, seed)
    if case["kind"] == "ensemble" and case["lattices"] * case["steps"] > 2000:
        return None  # one lattice at a time takes too long
    if case["kind"] == "gradient":
        ks = torch.full((case["nodes"],), cfg["capsules"][0]["ks"], dtype=torch.float64, device=dev, requires_grad=True)
        g = torch.tensor(float(cfg["body_force_x"]), dtype=torch.float64, device=dev, requires_grad=True)
        m = _Exact(cfg, dev, ks, g)
        for _ in range(case["steps"]):
            m.step()
        J = m.taylor()
        dks, dg = torch.autograd.grad(J, (ks, g))
        return {"J": np.float64(J.item()), "dJ_dg": np.float64(dg.item()), "dJ_dks": dks.cpu().numpy()}
    fields, nodes = [], []
    with torch.no_grad():
        for c in cfg if case["kind"] == "ensemble" else [cfg]:
            m = _Exact(c, dev)
            if not c["capsules"]:
                m.f = m.complete(_disturbed(case, c, seed, dev) - m.w[:, None, None])
            for _ in range(case["steps"] + (WARM if _restarts(case) else 0)):
                m.step()
            fields += [q.reshape(-1) for q in m.moments()]
            if c["capsules"]:
                uv = m.uv if case["mode"] == "dynamic" else m.first
                nodes += [q[m.cap == k].reshape(-1) for k in range(len(c["capsules"]))
                          for q in (m.x, m.x - m.d, uv)]
    out = {"fields": torch.cat(fields)} if len(fields) > 3 else {"rho": fields[0], "u": torch.cat(fields[1:])}
    if nodes:
        out["nodes"] = torch.cat(nodes)
    return out
