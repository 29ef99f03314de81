"""Kernel paths at the sizes where one takes over from another."""
import numpy as np
import pytest

from paper_1903_03356_amd import lbib
from paper_1903_03356_amd import workloads as wl
from tests.parity import log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", ["kinematic", "dynamic"])
@pytest.mark.parametrize("max_nodes", [100, 520])
def test_adjoint_patch_sums(max_nodes, mode):
    """Reverse IB kernel in FP32 on a patch of 39 x 36 cells or a little more:
    it sums its adjoints in FP64 where they take at most half the on-chip
    capacity (node capacity 100: 5984 cells), else in FP32 (node capacity 520:
    2624 cells); both against the FP64 run, with the FP32 gradient's bar of
    1e-3.  FP64 sums make the gradient repeat up to terms of 1e-16."""
    cfg = wl._base("patch", 128, 96, 0.8, 8, mode, 0, init_profile=wl.INIT_POISEUILLE,
                   body_force_x=wl.poiseuille_body_force(0.8, 96, 0.02))
    nodes = wl.circle_nodes(60.3, 45.2, 16.0, 100)
    nodes[:, 1] = 45.2 + 0.9 * (nodes[:, 1] - 45.2)
    cfg["capsules"] = [wl.capsule(nodes, wl.ks_from_ca(0.8, 0.02, 5e-2))]
    r8 = lbib.Sim(cfg).adjoint(30, mode=mode)
    cfg4 = dict(cfg, real_bytes=4)
    r4, again = (lbib.Sim(cfg4, max_nodes_capsule=max_nodes).adjoint(30, mode=mode)
                 for _ in range(2))
    k8, k4 = r8["dJ_dks"][0], r4["dJ_dks"][0]
    log(f"node capacity {max_nodes} {mode}: ks {np.abs(k4 - k8).max() / np.abs(k8).max():.1e}, "
        f"g {abs(r4['dJ_dg'] / r8['dJ_dg'] - 1):.1e}")
    assert np.abs(k4 - k8).max() <= 1e-3 * np.abs(k8).max()
    assert abs(r4["dJ_dg"] - r8["dJ_dg"]) <= 1e-3 * abs(r8["dJ_dg"])
    if max_nodes == 100:
        assert np.abs(again["dJ_dks"][0] - k4).max() <= 1e-6 * np.abs(k4).max()
        assert abs(again["dJ_dg"] - r4["dJ_dg"]) <= 1e-6 * abs(r4["dJ_dg"])


@pytest.mark.parametrize("nx,ny,real_bytes,periodic_y", [
    (1023, 480, 4, 0),   # two column blocks, the last one short by a column
    (545, 901, 4, 1),    # one column past a block of 544; both axes periodic
    (8191, 65, 4, 0),    # many blocks of few rows
    (70, 7001, 4, 0),    # one narrow block, wrapping within its halo
    (481, 601, 8, 0),    # FP64: one column past a block
    (40, 6500, 8, 1),
])
def test_two_steps_in_one_pass(nx, ny, real_bytes, periodic_y):
    """A capsule-free lattice large enough to take two steps per pass, at block
    edges and remainders, odd step counts: the same bits as one step per call."""
    cfg = wl._base("two", nx, ny, 0.7, real_bytes, "kinematic", 0, periodic_y=periodic_y,
                   u_bottom=-0.01, u_top=0.02, body_force_x=1e-6)
    if not periodic_y and nx == 1023:  # the storage reference of a Poiseuille channel
        cfg.update(u_bottom=0.0, u_top=0.0, init_profile=wl.INIT_POISEUILLE,
                   body_force_x=wl.poiseuille_body_force(0.7, ny, 0.02))
    f0 = wl.random_populations(nx, ny, seed=3, amp=0.01)
    a, b = lbib.Sim(cfg), lbib.Sim(cfg)
    for s in (a, b):
        s.set_pops(f0)
    for n in (5, 2, 1, 4):
        a.step(n)
        for _ in range(n):
            b.step(1)
        assert a.steps_done == b.steps_done
        np.testing.assert_array_equal(a.pops(), b.pops())
    np.testing.assert_array_equal(a.moments(), b.moments())
    assert a.check() == 0


def test_two_steps_under_capture():
    """A caller's graph of two steps repeats: its replays read and write the same
    buffers, so a recorded call takes single passes."""
    import torch
    cfg = wl._base("cap", 1024, 512, 0.7, 4, "kinematic", 0, u_top=0.02)
    f0 = wl.random_populations(1024, 512, seed=4, amp=0.01)
    st = torch.cuda.Stream()
    a, b = lbib.Sim(cfg, stream=st), lbib.Sim(cfg)
    for s in (a, b):
        s.set_pops(f0)
    st.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=st):
        a.step(2)
    for _ in range(3):
        graph.replay()
        torch.cuda.synchronize()
    b.step(6)
    np.testing.assert_array_equal(a.pops(), b.pops())


def _ellipse(cx, cy, a, b, n, angle=0.0):
    t = 2.0 * np.pi * (np.arange(n) + 0.5) / n
    x, y = a * np.cos(t), b * np.sin(t)
    c, s = np.cos(angle), np.sin(angle)
    return np.stack([cx + c * x - s * y, cy + s * x + c * y], axis=1)


def _fused_case(name, real_bytes, mode):
    """Lattice and capsules of one path of the capsule blocks' own grid step."""
    u, tau = 0.02, 0.8
    channel = dict(init_profile=wl.INIT_POISEUILLE)
    if name == "open":  # an end column and a wall row in the ring
        cfg = wl.open_channel(96, 64, tau, u, real_bytes=real_bytes, mode=mode,
                              init_profile=wl.INIT_INLET)
        shapes = [_ellipse(9.0, 12.0, 5.5, 6.0, 40), _ellipse(86.0, 40.0, 6.0, 6.0, 40)]
    elif name == "box":  # both axes wrap
        cfg = wl.periodic_box(70, 45, tau, u0=(u, -u), real_bytes=real_bytes, mode=mode)
        shapes = [_ellipse(2.0, 43.5, 6.0, 5.0, 40), _ellipse(35.0, 20.0, 8.0, 5.0, 48, 0.5)]
    elif name == "contact":  # three in contact, one of them over the wrap
        cfg = wl.periodic_box(70, 45, tau, u0=(u, -u), real_bytes=real_bytes, mode=mode)
        cfg["contact_cutoff"] = 2.0
        shapes = [_ellipse(2.0, 20.0, 6.0, 5.0, 40), _ellipse(14.6, 20.0, 5.5, 6.0, 40),
                  _ellipse(59.2, 21.0, 5.5, 6.0, 40)]
    elif name == "bands":  # FP64: the ring of a large capsule in several bands of rows
        cfg = wl._base(name, 160, 128, tau, real_bytes, mode, 0,
                       body_force_x=wl.poiseuille_body_force(tau, 128, u), **channel)
        shapes = [_ellipse(80.3, 60.2, 22.0, 21.0, 120)]
    elif name == "direct":  # FP64: a patch so wide that no row of the ring fits
        cfg = wl._base(name, 400, 48, tau, real_bytes, mode, 0,
                       body_force_x=wl.poiseuille_body_force(tau, 48, u), **channel)
        shapes = [_ellipse(200.0, 22.0, 140.0, 3.0, 120)]
    else:  # walls: moving walls, one capsule on each, patches over the wall rows and the wrap
        cfg = wl._base(name, 130, 40, tau, real_bytes, mode, 0, u_bottom=-u, u_top=u,
                       init_profile=wl.INIT_COUETTE)
        shapes = [_ellipse(3.0, 9.2, 6.0, 6.0, 40), _ellipse(64.0, 29.9, 9.0, 6.0, 60)]
    cfg["capsules"] = [wl.capsule(p, 0.05, 0.0, 1.0, 1.2) for p in shapes]
    return cfg


@pytest.mark.parametrize("mode", ["dynamic", "kinematic"])
@pytest.mark.parametrize("name,real_bytes", [("walls", 4), ("walls", 8), ("box", 4), ("open", 4),
                                             ("open", 8), ("bands", 8), ("direct", 8),
                                             ("contact", 4), ("contact", 8)])
def test_one_launch_per_step(name, real_bytes, mode):
    """A step as one launch (the automatic schedule of a single lattice): the
    same bits as a grid and an IB launch per step, also after the nodes were
    moved by hand (the patch box of the last launch does not fit) and across a
    change of schedule between calls."""
    cfg = _fused_case(name, real_bytes, mode)
    a, b = lbib.Sim(cfg), lbib.Sim(cfg)
    b.set_overlap(False)

    def same():
        np.testing.assert_array_equal(a.pops(), b.pops())
        np.testing.assert_array_equal(a.force(), b.force())
        for c in range(len(a.nv)):
            np.testing.assert_array_equal(np.stack(a.capsule(c)), np.stack(b.capsule(c)))

    for n in (1, 6):
        a.step(n)
        b.step(n)
        same()
    x, xp, uv = a.capsule(0)
    shift = np.array([0.0, 2.0]) if name != "direct" else np.array([2.0, 0.0])
    for s in (a, b):
        s.set_capsule(0, x + shift, xp + shift, uv)
        s.step(3)
    same()
    a.set_overlap(False)
    b.set_overlap(None)
    for s in (a, b):
        s.step(4)
    same()
    assert a.check() == b.check()


def _pair_case(name, real_bytes, mode):
    """Lattices past the size from which two steps with capsules share a pass."""
    u, tau = 0.02, 0.8

    def lattice(nx, ny, shapes, **kw):
        cfg = wl._base(name, nx, ny, tau, real_bytes, mode, 0, **kw)
        cfg["capsules"] = [wl.capsule(p, 0.05, 0.0, 1.0, 1.2) for p in shapes]
        return cfg

    if name == "box":  # both axes wrap: a capsule across the corner, one across rows of blocks
        n = 2050 if real_bytes == 4 else 1450
        return lattice(n, n - 3, [_ellipse(2.0, n - 4.5, 6.0, 5.0, 40),
                                  _ellipse(500.0, 66.0, 8.0, 5.0, 48, 0.5)],
                       periodic_y=1, init_profile=wl.INIT_UNIFORM, init_u=(u, -u))
    if name == "channel":  # capsules beside the walls and each other, over the wrap
        return lattice(4097, 1100, [_ellipse(3.0, 9.2, 6.0, 6.0, 40),
                                    _ellipse(64.0, 1089.0, 9.0, 6.0, 60),
                                    _ellipse(543.0, 500.0, 7.0, 7.0, 50),
                                    _ellipse(559.5, 501.0, 7.0, 7.0, 50)],
                       init_profile=wl.INIT_POISEUILLE,
                       body_force_x=wl.poiseuille_body_force(tau, 1100, u))
    walls = dict(u_bottom=-u, u_top=u, init_profile=wl.INIT_COUETTE)
    n = 1 if real_bytes == 4 else 2
    return [lattice(1500 // n, 1100, [_ellipse(250.0, 30.0, 7.0, 6.0, 40)], **walls),
            lattice(40, 33, [_ellipse(20.0, 16.0, 5.0, 5.0, 30)], **walls),
            lattice(1457 // n, 1300, [_ellipse(300.0, 900.0, 7.0, 6.0, 40),
                                      _ellipse(2.0, 9.5, 6.0, 6.0, 40)], **walls),
            lattice(257, 64, [_ellipse(255.0, 30.0, 8.0, 6.0, 40)], periodic_y=1, init_profile=wl.INIT_UNIFORM,
                    init_u=(u, u)),
            lattice(513, 1200, [_ellipse(511.0, 600.0, 8.0, 6.0, 40)], **walls)]


@pytest.mark.parametrize("mode", ["dynamic", "kinematic"])
@pytest.mark.parametrize("real_bytes", [4, 8])
@pytest.mark.parametrize("name", ["box", "channel", "batch"])
def test_two_steps_with_capsules(name, real_bytes, mode):
    """Two steps with capsules in one pass (the automatic schedule of large
    lattices and batches): the same bits as a grid and an IB launch per step,
    also for odd counts and across a change of schedule between calls."""
    cfg = _pair_case(name, real_bytes, mode)
    make = lbib.Batch if isinstance(cfg, list) else lbib.Sim
    a, b = make(cfg), make(cfg)
    b.set_overlap(False)

    def same():
        for i in range(len(cfg) if isinstance(cfg, list) else 1):
            np.testing.assert_array_equal(a.pops(i), b.pops(i))
            np.testing.assert_array_equal(a.force(i), b.force(i))
        for c in range(len(a.nv)):
            np.testing.assert_array_equal(np.stack(a.capsule(c)), np.stack(b.capsule(c)))

    for n in (2, 5, 1, 4):
        a.step(n)
        b.step(n)
        same()
    a.set_overlap(False)
    b.set_overlap(None)
    for s in (a, b):
        s.step(4)
    same()
    if not isinstance(cfg, list) and real_bytes == 4:
        a.set_overlap(True)
        for s in (a, b):
            s.step(3)
        same()
    assert a.check() == 0 and b.check() == 0


@pytest.mark.parametrize("mode", ["dynamic", "kinematic"])
def test_capsules_under_capture(mode):
    """A caller's graph of two steps, recorded after steps of the automatic
    schedule, repeats with the caller's own steps between its replays."""
    import torch
    cfg = _fused_case("walls", 4, mode)
    st = torch.cuda.Stream()
    a, b = lbib.Sim(cfg, stream=st), lbib.Sim(cfg)
    b.set_overlap(False)
    a.step(3)
    b.step(3)
    st.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=st):
        a.step(2)
    for _ in range(3):
        graph.replay()
        torch.cuda.synchronize()
        a.step(4)
        b.step(6)
        np.testing.assert_array_equal(a.pops(), b.pops())
        np.testing.assert_array_equal(np.stack(a.capsule(0)), np.stack(b.capsule(0)))


def _contact_oracle(shapes, L, cutoff):
    """Eq. 27 on every node in FP64, a periodic box of side L."""
    normals = []
    for x in shapes:
        e = np.roll(x, -1, axis=0) - x
        e /= np.linalg.norm(e, axis=1, keepdims=True)
        n = np.stack([e[:, 1], -e[:, 0]], 1)
        n = n + np.roll(n, 1, axis=0)
        normals.append(-n / np.linalg.norm(n, axis=1, keepdims=True))
    out = []
    for c, x in enumerate(shapes):
        other = np.concatenate([s for o, s in enumerate(shapes) if o != c])
        d = x[:, None] - other[None]
        d -= L * np.rint(d / L)
        d = np.sqrt((d ** 2).sum(-1))
        mag = np.where((d < cutoff) & (d > 0), (1e-4 / (8 * np.sqrt(2.0))) / np.maximum(d, 1e-9) ** 2.5,
                       0.0)
        out.append(mag.sum(1)[:, None] * normals[c])
    return out


@pytest.mark.parametrize("name,real_bytes,tol", [
    ("neighbours", 8, 1e-10),  # 1440 nodes of eight neighbours: staged in two rounds
    ("many", 8, 1e-10),        # 196 capsules: two rounds of records
    ("large", 4, 2e-6),        # 600 nodes: more than threads in a block
])
def test_contact_rounds(name, real_bytes, tol):
    """The contact force where its kernel goes in several rounds, against an FP64
    sum over all nodes.  The membranes are at rest with a stiffness that leaves
    at most 1e-17 beside the force; FP64: positions to 1e-14 on distances of 0.5
    and more, FP32: the force is stored in 24 bits."""
    L = 128
    if name == "neighbours":
        shapes = [_ellipse(20.0 + 18.0 * i, 20.0 + 18.0 * j, 8.6, 8.6, 180) for i in range(3)
                  for j in range(3)]
    elif name == "many":
        p = L / 14.0
        shapes = [_ellipse((i + 0.5) * p, (j + 0.5) * p, 4.0, 4.0, 16) for i in range(14)
                  for j in range(14)]
    else:
        shapes = [_ellipse(40.0, 40.0, 15.0, 12.0, 600), _ellipse(70.5, 40.0, 15.0, 12.0, 600)]
    cfg = wl._base("contact", L, L, 0.8, real_bytes, "kinematic", 0, periodic_y=1)
    cfg["contact_cutoff"] = 2.0
    cfg["capsules"] = [wl.capsule(p, 1e-17, 0.0, 0.0) for p in shapes]
    s = lbib.Sim(cfg)
    s.step(1)
    want = _contact_oracle(shapes, L, 2.0)
    scale = max(np.abs(f).max() for f in want)
    err = max(np.abs(s.capsule_force(c) - want[c]).max() for c in range(len(shapes)))
    log(f"contact {name}: force {scale:.1e}, error {err / scale:.1e}")
    assert scale > 1e-6 and err <= tol * scale


def test_far_pass_waits_for_fp64_capsules():
    """The split schedule of a large FP64 lattice: its IB launch cannot run beside
    a far pass that waits for it, so the far pass waits on its queue; same bits as
    a single pass, no wait given up."""
    cfg = wl._base("far", 4096, 2049, 0.8, 8, "dynamic", 0, u_bottom=-0.02, u_top=0.02,
                   init_profile=wl.INIT_COUETTE)
    cfg["capsules"] = [wl.capsule(_ellipse(100.0 + 480.0 * i, 200.0 + 200.0 * i, 8.0, 6.0, 60),
                                  0.05, 0.0, 1.0, 1.2) for i in range(8)]
    a, b = lbib.Sim(cfg), lbib.Sim(cfg)
    a.set_overlap(True)
    b.set_overlap(False)
    for s in (a, b):
        s.step(6)
    assert a.check() == 0
    np.testing.assert_array_equal(a.force(), b.force())
    for c in range(8):
        np.testing.assert_array_equal(np.stack(a.capsule(c)), np.stack(b.capsule(c)))


@pytest.mark.parametrize("real_bytes", [4, 8])
@pytest.mark.parametrize("name", ["walls", "box", "open", "bands"])
def test_populations_on_the_device(name, real_bytes):
    """The nine planes set and read in one launch (device buffers) are those set
    and read one by one (host buffers)."""
    import torch
    cfg = dict(_fused_case(name, real_bytes, "dynamic"), capsules=[])
    f0 = wl.random_populations(cfg["nx"], cfg["ny"], seed=5, amp=0.01)
    a, b = lbib.Sim(cfg), lbib.Sim(cfg)
    a.set_state(lbib.F_POPS, f0)
    b.set_state(lbib.F_POPS, torch.from_numpy(np.ascontiguousarray(f0)).cuda())
    for n in (0, 1, 2):
        a.step(n)
        b.step(n)
        for what in (lbib.F_POPS, lbib.F_POPS_DEV):
            out = torch.empty(f0.shape, dtype=torch.float64, device="cuda")
            b.get_state(what, 0, out=out)
            np.testing.assert_array_equal(out.cpu().numpy(), a.get_state(what, 0))


def test_autotune_between_steps():
    """Trial passes between two Dynamic calls of a batch, the first of which spread
    the forcing of the second ahead: the same bits as without them."""
    cfg = _pair_case("batch", 4, "dynamic")
    a, b = lbib.Batch(cfg), lbib.Batch(cfg)
    for s in (a, b):
        s.step(2)
    a.autotune(1)
    for s in (a, b):
        s.step(2)
    for i in range(len(cfg)):
        np.testing.assert_array_equal(a.pops(i), b.pops(i))
        np.testing.assert_array_equal(a.force(i), b.force(i))
    np.testing.assert_array_equal(np.stack(a.capsule(0)), np.stack(b.capsule(0)))


def test_moments_of_a_large_lattice():
    """From 2^20 cells the moments take the force of active segments only: on a
    lattice with capsules, the velocity that the populations and the whole force
    field give (FP64; sums of a dozen terms of at most 1: 1e-14)."""
    cfg = _pair_case("channel", 8, "dynamic")
    s = lbib.Sim(cfg)
    s.step(3)
    rho, ux, uy = s.moments()
    f, F = s.pops(), s.force()
    ex = np.array([0, 1, 0, -1, 0, 1, -1, -1, 1.0])
    ey = np.array([0, 0, 1, 0, -1, 1, 1, -1, -1.0])
    assert np.abs(F[1]).max() > 0
    np.testing.assert_allclose(rho, f.sum(0), rtol=0, atol=1e-14)
    inner = slice(1, -1)
    for u, e, k in ((ux, ex, 0), (uy, ey, 1)):
        want = (np.tensordot(e, f, 1) + 0.5 * F[k]) / f.sum(0)
        np.testing.assert_allclose(u[inner], want[inner], rtol=0, atol=1e-14)


def _recorded_case(name, mode="dynamic"):
    """Lattices of the schedules that exchange buffers or force levels."""
    if name == "fused":
        return _fused_case("walls", 4, mode)
    if name == "contact":
        return _fused_case("contact", 8, mode)
    if name == "pair":
        return _pair_case("channel", 4, mode)
    return wl._base("two", 1024, 512, 0.7, 4, "kinematic", 0, u_top=0.02,
                    init_profile=wl.INIT_COUETTE)


def _device_like(sim, what, cap=0):
    import torch
    nx, ny = sim.dims[0]
    shape = {lbib.F_POPS: (9, ny, nx), lbib.F_MOMENTS: (3, ny, nx), lbib.F_FORCE: (2, ny, nx),
             lbib.C_STATE: (3, sim.nv[cap] if sim.nv else 1, 2)}[what]
    return torch.zeros(shape, dtype=torch.float64, device="cuda")


@pytest.mark.parametrize("name,mode", [("fused", "dynamic"), ("fused", "kinematic"),
                                       ("contact", "kinematic"), ("pair", "dynamic"), ("two", "kinematic")])
def test_recorded_read_out(name, mode):
    """A caller's graph of read-outs, recorded after steps of the automatic schedule,
    reads the state after every even number of the caller's own steps."""
    import torch
    cfg = _recorded_case(name, mode)
    st = torch.cuda.Stream()
    a, b = lbib.Sim(cfg, stream=st), lbib.Sim(cfg)
    b.set_overlap(False)
    whats = [lbib.F_POPS, lbib.F_MOMENTS, lbib.F_FORCE] + ([lbib.C_STATE] if a.nv else [])
    out = [_device_like(a, w) for w in whats]
    torch.cuda.synchronize()
    a.step(4)
    b.step(4)
    st.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=st):
        for w, o in zip(whats, out):
            a.get_state(w, 0, out=o)
    for n in (0, 2, 4, 6):
        a.step(n)
        b.step(n)
        graph.replay()
        torch.cuda.synchronize()
        for w, o in zip(whats, out):
            np.testing.assert_array_equal(o.cpu().numpy(), b.get_state(w, 0))


@pytest.mark.parametrize("name,mode", [("fused", "dynamic"), ("fused", "kinematic"), ("pair", "dynamic"),
                                       ("two", "kinematic")])
@pytest.mark.parametrize("before", [0, 4])
def test_recorded_restart(name, mode, before):
    """A caller's graph that restores a saved state, recorded before the first step or
    after steps of the automatic schedule (the Dynamic one spreads the forcing of the
    coming call ahead), with steps between the recording and its first replay."""
    import torch
    cfg = _recorded_case(name, mode)
    st = torch.cuda.Stream()
    a, b = lbib.Sim(cfg, stream=st), lbib.Sim(cfg)
    b.set_overlap(False)
    whats = [lbib.F_POPS] + ([lbib.C_STATE] if a.nv else [])
    saved = [_device_like(a, w) for w in whats]
    src = lbib.Sim(cfg)
    src.step(2)
    for w, x in zip(whats, saved):
        src.get_state(w, 0, out=x)
    torch.cuda.synchronize()
    a.step(before)
    b.step(before)
    st.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=st):
        for w, x in zip(whats, saved):
            a.set_state(w, x, 0)

    def same():
        np.testing.assert_array_equal(a.pops(), b.pops())
        np.testing.assert_array_equal(a.force(), b.force())
        if a.nv:
            np.testing.assert_array_equal(np.stack(a.capsule(0)), np.stack(b.capsule(0)))

    a.step(2)
    b.step(2)
    same()
    for _ in range(3):
        graph.replay()
        for w, x in zip(whats, saved):
            b.set_state(w, x, 0)
        for s in (a, b):
            s.step(4)
        torch.cuda.synchronize()
        same()


def test_steps_after_a_recording_not_replayed():
    """Steps recorded while a forcing is spread ahead drop it in the graph; the
    caller's next step, before any replay, starts from a clean level all the same."""
    import torch
    cfg = _fused_case("walls", 4, "dynamic")
    st = torch.cuda.Stream()
    a, b = lbib.Sim(cfg, stream=st), lbib.Sim(cfg)
    b.set_overlap(False)
    a.step(4)
    b.step(4)
    st.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=st):
        a.step(2)
    for n in (2, 4):
        a.step(n)
        b.step(n)
        np.testing.assert_array_equal(a.pops(), b.pops())
        np.testing.assert_array_equal(np.stack(a.capsule(0)), np.stack(b.capsule(0)))
    for _ in range(3):
        graph.replay()
        b.step(2)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(a.pops(), b.pops())
        np.testing.assert_array_equal(np.stack(a.capsule(0)), np.stack(b.capsule(0)))


@pytest.mark.parametrize("overlap", [None, True, "ahead"])
def test_large_lattice_under_capture(overlap):
    """A caller's graph of steps of a lattice past the size of the overlapped schedule
    (its far pass waits inside from 2^23 cells), asked for or not, or asked for until
    just before ("ahead": it left the forcing of the next step spread): every replay
    computes its own near regions, also after the capsules were moved."""
    import torch
    cfg = wl._base("cap", 4096, 2049, 0.8, 4, "dynamic", 0, u_bottom=-0.02, u_top=0.02,
                   init_profile=wl.INIT_COUETTE)
    cfg["capsules"] = [wl.capsule(_ellipse(100.0 + 480.0 * i, 200.0 + 200.0 * i, 8.0, 6.0, 60),
                                  0.05, 0.0, 1.0, 1.2) for i in range(8)]
    st = torch.cuda.Stream()
    a, b = lbib.Sim(cfg, stream=st), lbib.Sim(cfg)
    a.set_overlap(True if overlap == "ahead" else overlap)
    b.set_overlap(False)
    a.step(2)
    b.step(2)
    if overlap == "ahead":
        a.set_overlap(False)
    st.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=st):
        a.step(2)
    for k in range(4):
        graph.replay()
        b.step(2)
        torch.cuda.synchronize()
        if k == 1:  # far enough for other rows and segments, past what a stale map holds
            for c in range(8):
                x, xp, uv = b.capsule(c)
                for s in (a, b):
                    s.set_capsule(c, x + [70.0, 20.0], xp + [70.0, 20.0], uv)
        if k == 2:  # the caller's own steps between
            a.step(2)
            b.step(2)
    np.testing.assert_array_equal(a.pops(), b.pops())
    np.testing.assert_array_equal(a.force(), b.force())
    for c in range(8):
        np.testing.assert_array_equal(np.stack(a.capsule(c)), np.stack(b.capsule(c)))
    assert a.check() == b.check() == 0


def _grid_of_capsules(nx, ny, cols, rows, a=8.0, b=6.0):
    return [wl.capsule(_ellipse((i + 0.5) * nx / cols, 8 + (j + 0.5) * (ny - 16) / rows, a, b, 60),
                       0.05, 0.0, 1.0, 1.2) for j in range(rows) for i in range(cols)]


@pytest.mark.parametrize("ny,cols,rows", [(2049, 8, 8), (2049, 13, 5), (4096, 32, 16)])
def test_overlap_of_many_capsules(ny, cols, rows):
    """The split schedule of a large FP32 lattice at and past the number of capsules
    up to which its far pass waits inside: no wait given up, the bits of a single pass."""
    cfg = wl._base("far", 4096, ny, 0.8, 4, "dynamic", 0, u_bottom=-0.02, u_top=0.02,
                   init_profile=wl.INIT_COUETTE)
    cfg["capsules"] = _grid_of_capsules(4096, ny, cols, rows)
    a, b = lbib.Sim(cfg), lbib.Sim(cfg)
    a.set_overlap(True)
    b.set_overlap(False)
    for s in (a, b):
        s.step(5)
    assert a.check() == b.check() == 0
    np.testing.assert_array_equal(a.force(), b.force())
    for c in range(0, cols * rows, 7):
        np.testing.assert_array_equal(np.stack(a.capsule(c)), np.stack(b.capsule(c)))


@pytest.mark.parametrize("real_bytes", [4, 8])
def test_timed_steps_take_a_launch_each(real_bytes):
    """Kernel timing of a capsule-free lattice that takes two steps per pass when it is
    off: one timed grid launch per step, also for odd counts; the same bits either way,
    and with the schedule of one launch per step asked for."""
    cfg = wl._base("two", 1024, 512, 0.7, real_bytes, "kinematic", 0, u_top=0.02,
                   init_profile=wl.INIT_COUETTE)
    a, b, c = lbib.Sim(cfg), lbib.Sim(cfg), lbib.Sim(cfg)
    a.set_timing(True)
    c.set_overlap(False)
    for n in (4, 3):
        for s in (a, b, c):
            s.step(n)
    t = a.get_timing()
    assert t["grid_launches"] == 7 and t["ib_launches"] == 0
    a.set_timing(False)
    for s in (a, b, c):
        s.step(2)
    assert a.get_timing()["grid_launches"] == 0
    np.testing.assert_array_equal(a.pops(), b.pops())
    np.testing.assert_array_equal(a.pops(), c.pops())


@pytest.mark.parametrize("nx,ny,real_bytes,ends", [
    (1601, 1680, 4, "walls"), (1601, 1681, 4, "walls"),   # both buffers just within and just
    (1024, 1285, 8, "walls"), (1024, 1286, 8, "walls"),   # past 192 MiB
    (1024, 1285, 8, "open"), (1024, 1286, 8, "open"),
])
def test_single_passes_around_the_load_rule(nx, ny, real_bytes, ends):
    """A launch per grid step where the kernel turns from plain to streaming loads: the
    same bits as two steps per pass, and (open ends, a capsule) as one launch per step."""
    if ends == "open":
        cfg = wl.open_channel(nx, ny, 0.8, 0.02, real_bytes=real_bytes, mode="dynamic",
                              init_profile=wl.INIT_INLET)
        cfg["capsules"] = [wl.capsule(wl.circle_nodes(80.3, 70.6, 8.0, 60), 0.05, 0.0, 1.0, 1.2)]
    else:
        cfg = wl._base("one", nx, ny, 0.7, real_bytes, "kinematic", 0, u_top=0.02)
    f0 = wl.random_populations(nx, ny, seed=6, amp=0.01)
    a, b = lbib.Sim(cfg), lbib.Sim(cfg)
    b.set_overlap(False)
    for s in (a, b):
        s.set_pops(f0)
    for n in (4, 1):
        a.step(n)
        b.step(n)
        np.testing.assert_array_equal(a.pops(), b.pops())
    assert a.check() == b.check()


def _step_us(sim, steps, calls=1):
    """Microseconds a step, the least of seven timings."""
    import torch
    best = 1e30
    for i in range(8):
        e0, e1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        e0.record()
        for _ in range(calls):
            sim.step(steps)
        e1.record()
        torch.cuda.synchronize()
        if i:
            best = min(best, 1e3 * e0.elapsed_time(e1) / (steps * calls))
    return best


def _default_against_serial(cfg, steps, bar):
    """The automatic schedule takes at most `bar` times as long as one IB and one grid
    launch per step, in the same buffers (two contexts' can differ by 5 %: their memory
    lies elsewhere)."""
    s = (lbib.Batch if isinstance(cfg, list) else lbib.Sim)(cfg)
    for _ in range(3):  # (a machine that stalls in one of them)
        t = {}
        for overlap in (None, False):
            s.set_overlap(overlap)
            t[overlap] = _step_us(s, steps)
        log(f"{t[None]:.1f} us a step, serial {t[False]:.1f}")
        if t[None] <= bar * t[False]:
            return
    assert t[None] <= bar * t[False]


@pytest.mark.parametrize("name,real_bytes", [("grid", 4), ("capsules", 4), ("batch", 4)])
def test_narrow_lattices_take_single_passes(name, real_bytes):
    """Rows of a segment or less: two steps in one pass would take 1.2 (batch) to 1.9
    times as long as single ones (the bar: one route timed twice, to 6 %)."""
    def lattice(nx, ny, caps):
        cfg = wl._base("narrow", nx, ny, 0.8, real_bytes, "kinematic", 0,
                       init_profile=wl.INIT_POISEUILLE,
                       body_force_x=wl.poiseuille_body_force(0.8, ny, 0.02))
        cfg["capsules"] = [wl.capsule(_ellipse(0.5 * nx, ny * (i + 1.0) / (caps + 1), 6.0, 6.0, 50),
                                      0.01, 0.0, 1.0, 1.0) for i in range(caps)]
        return cfg
    cfg = {"grid": lambda: lattice(16, 27306, 0), "capsules": lambda: lattice(48, 70000, 4),
           "batch": lambda: [lattice(40, 47, i % 200 == 0) for i in range(2500)]}[name]()
    _default_against_serial(cfg, 20, 1.06)


@pytest.mark.parametrize("mode", ["dynamic", "kinematic"])
@pytest.mark.parametrize("name,real_bytes,mid,large", [("bands", 8, 13.0, 22.0), ("direct", 8, 0.0, 140.0),
                                                       ("bands", 4, 21.0, 38.0)])
def test_patch_that_outgrew_its_launch(name, real_bytes, mid, large, mode):
    """The patch's own grid step in bands of rows, and of a patch so wide that no row of
    its ring fits: shapes that the schedule of one launch per step is not chosen for
    are reached by deforming a capsule that it is chosen for.  The same bits as a grid
    and an IB launch per step."""
    u, tau = 0.02, 0.8
    nx, ny = (400, 48) if name == "direct" else (160, 128)
    cfg = wl._base(name, nx, ny, tau, real_bytes, mode, 0, init_profile=wl.INIT_POISEUILLE,
                   body_force_x=wl.poiseuille_body_force(tau, ny, u))
    c = (200.0, 22.0) if name == "direct" else (80.3, 60.2)
    # a star: a small patch, and a perimeter that sizes the LDS for a large one
    n = 120
    t = 2.0 * np.pi * (np.arange(n) + 0.5) / n
    r = 6.0 * (1.0 + 0.5 * np.cos(12 * t))
    star = np.stack([c[0] + r * np.cos(t), c[1] + r * np.sin(t)], 1)
    cfg["capsules"] = [wl.capsule(star, 1e-6, 0.0, 0.0, 1.2)]
    a, b = lbib.Sim(cfg), lbib.Sim(cfg)
    b.set_overlap(False)

    def same():
        np.testing.assert_array_equal(a.pops(), b.pops())
        np.testing.assert_array_equal(a.force(), b.force())
        np.testing.assert_array_equal(np.stack(a.capsule(0)), np.stack(b.capsule(0)))

    for s in (a, b):
        s.step(2)
    same()
    for size in (mid, large):
        if not size:
            continue
        x = _ellipse(*c, size, 3.0 if name == "direct" else size - 1.0, n)
        for s in (a, b):
            s.set_capsule(0, x, x, np.zeros_like(x))
            s.step(3)
        same()
    assert a.check() == b.check()


@pytest.mark.parametrize("nx,ny,real_bytes,radius,caps,mode", [
    (512, 200, 8, 26.0, 1, "kinematic"),    # dozens of bands of rows: 3.9 times as long
    (512, 200, 8, 20.0, 1, "kinematic"),    # 4 bands: 1.4
    (512, 200, 8, 2.3, 1, "kinematic"),     # a ring that the LDS of a tiny patch does not hold: 1.3
    (512, 200, 4, 40.0, 1, "kinematic"),    # 2.5
    (1024, 512, 4, 40.0, 6, "dynamic"),     # 2.1
    (1500, 1400, 8, 28.0, 6, "dynamic"),    # two steps per pass: 1.8
])
def test_large_capsules_take_two_launches(nx, ny, real_bytes, radius, caps, mode):
    """Capsules whose patch does not step well by itself (the factors: the schedules of
    one launch per step and of two steps per pass, where they do not suit); the bar:
    one route timed twice, to 6 %."""
    n = int(2 * np.pi * radius / 0.75) + 1
    cfg = wl._base("large", nx, ny, 0.8, real_bytes, mode, 0, init_profile=wl.INIT_POISEUILLE,
                   body_force_x=wl.poiseuille_body_force(0.8, ny, 0.02))
    cfg["capsules"] = [wl.capsule(_ellipse(nx * (i + 0.5) / caps, 0.5 * ny, radius, radius, n),
                                  wl.ks_from_ca(0.8, 0.02, 5e-2), 0.0, 1.0, 1.2) for i in range(caps)]
    _default_against_serial(cfg, 15, 1.06)


@pytest.mark.parametrize("kind,n,real_bytes", [("open", 2304, 4), ("contact", 3000, 4), ("contact", 2600, 8)])
def test_large_lattices_take_two_launches(kind, n, real_bytes):
    """Open channels and the contact force on lattices past the cache, where one launch
    per step takes 1.07 to 1.11 times as long as two; the bar: one route timed twice, to
    5 %."""
    if kind == "open":
        cfg = wl.open_channel(n, n, 0.8, 0.02, real_bytes=real_bytes, mode="dynamic",
                              init_profile=wl.INIT_INLET)
    else:
        cfg = wl._base("contact", n, n, 0.8, real_bytes, "kinematic", 0, init_profile=wl.INIT_POISEUILLE,
                       body_force_x=wl.poiseuille_body_force(0.8, n, 0.02))
        cfg["contact_cutoff"] = 2.0
    cfg["capsules"] = _grid_of_capsules(n, n, 4, 4)
    _default_against_serial(cfg, 15, 1.05)


@pytest.mark.parametrize("name", ["lattice", "small", "batch"])
def test_many_capsules_take_two_launches(name):
    """Lattices full of capsules, whose own steps and near cells cost more than the
    passes they spare: 1.3 to 1.6 times as long as one IB and one grid launch per step;
    the bar: one route timed twice, to 6 %."""
    def lattice(nx, ny, cols, rows):
        cfg = wl._base("many", nx, ny, 0.8, 4, "dynamic", 0, init_profile=wl.INIT_POISEUILLE,
                       body_force_x=wl.poiseuille_body_force(0.8, ny, 0.02))
        cfg["capsules"] = _grid_of_capsules(nx, ny, cols, rows)
        return cfg
    cfg = {"lattice": lambda: lattice(2048, 2048, 32, 32), "small": lambda: lattice(1024, 1024, 32, 25),
           "batch": lambda: [lattice(400, 100, 6, 2) for _ in range(128)]}[name]()
    _default_against_serial(cfg, 10, 1.06)


@pytest.mark.parametrize("mode", ["dynamic", "kinematic"])
@pytest.mark.parametrize("name", ["batch", "bands"])
def test_two_steps_with_capsules_fp64(name, mode):
    """Two steps in one pass in FP64: a batch past the size from which it takes them, and
    capsules whose rings go in three bands of rows on a lattice large enough for that;
    the same bits as a grid and an IB launch per step."""
    if name == "batch":
        cfg = [dict(c, real_bytes=8) for c in _pair_case("batch", 4, mode)]
    else:
        cfg = wl._base(name, 1450, 1447, 0.8, 8, mode, 0, periodic_y=1, init_profile=wl.INIT_UNIFORM,
                       init_u=(0.02, -0.02))
        cfg["capsules"] = [wl.capsule(_ellipse(5.0, 1440.0, 18.0, 17.0, 150), 0.05, 0.0, 1.0, 1.2),
                           wl.capsule(_ellipse(700.0, 300.0, 18.0, 16.0, 150), 0.05, 0.0, 1.0, 1.2)]
    make = lbib.Batch if isinstance(cfg, list) else lbib.Sim
    a, b = make(cfg), make(cfg)
    b.set_overlap(False)
    for n in (3, 4):
        a.step(n)
        b.step(n)
        for i in range(len(cfg) if isinstance(cfg, list) else 1):
            np.testing.assert_array_equal(a.pops(i), b.pops(i))
            np.testing.assert_array_equal(a.force(i), b.force(i))
        for c in range(len(a.nv)):
            np.testing.assert_array_equal(np.stack(a.capsule(c)), np.stack(b.capsule(c)))
    assert a.check() == b.check() == 0
