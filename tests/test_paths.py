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
