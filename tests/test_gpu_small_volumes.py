"""GPU parity of the small-volume kernel (FP64 volumes of at most 512 segments
and nodes): one force evaluation, one step, and bursts in the persistent launch,
at sizes around its edges (one segment, a wavefront of sources more or less,
the largest volume, more target points than one round holds), with nodes of
degree 1 and above 2, two slip planes at a node, pinned nodes and free nodes
without segments.

Tolerances: the library's stated 1e-10 against the FP64 oracle (normwise) and
1e-12 between the persistent launch and the step graph.
"""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2005_02498_amd as dd
from gpu_util import MAT, normwise
from paper_2005_02498_amd import workloads as W

pytestmark = pytest.mark.gpu

SIG = np.array([2e7, -3e7, 5e7, 1e7, -2e7, 4e7])


def _network(seed, n_segs, hub=0):
    """Chains of random FCC segments: n_segs segments, `hub` of which all start
    at one node, one free node without segments, every fifth node pinned."""
    rng = np.random.default_rng(seed)
    x = [rng.uniform(0.0, 800.0, 3)]
    seg, bur, nor = [], [], []
    last = 0
    for s in range(n_segs):
        system = int(rng.integers(0, 12)) if s % 7 == 0 or s < hub else system
        p, d = divmod(system, 3)
        n = W.PLANE_NORMALS[p]
        step = np.cross(n, rng.normal(size=3))
        step *= rng.uniform(15.0, 60.0) / np.linalg.norm(step)
        start = 0 if s < hub else last
        x.append(x[start] + step)
        last = len(x) - 1
        seg.append((start, last) if rng.random() < 0.8 else (last, start))
        bur.append(W.SLIP_DIRS[p, d] * rng.choice([-1.0, 1.0]))
        nor.append(n)
    x.append(rng.uniform(0.0, 800.0, 3))
    x = np.ascontiguousarray(np.array(x).T)
    pinned = np.zeros(x.shape[1], np.uint8)
    pinned[4::5] = 1
    return W.Instance(x, np.ascontiguousarray(np.array(seg, np.int32).T), np.ascontiguousarray(np.array(bur).T),
                      np.ascontiguousarray(np.array(nor).T), pinned, SIG, 8e9)


def _dev(i):
    d = torch.device("cuda:0")
    return [torch.tensor(a, device=d) for a in (i.x, i.seg_nodes, i.burgers, i.normal, i.pinned)]


@pytest.mark.parametrize("n_segs,hub,Q", [(1, 0, 2), (2, 0, 16), (63, 5, 3), (64, 0, 2), (65, 64, 1), (200, 3, 5),
                                          (256, 0, 4), (257, 9, 2), (449, 0, 3), (510, 40, 2)])
def test_one_step_vs_oracle(n_segs, hub, Q):
    inst = _network(n_segs, n_segs, hub)
    F = O.nodal_forces(inst.x, inst.seg_nodes, inst.burgers, inst.sigma_app, W.MU, W.NU, W.CORE_A, Q)
    xn, v = O.glide_step(inst.x, F, inst.seg_nodes, inst.normal, inst.pinned, W.DRAG_B, W.DT)
    x, sn, b, n, p = _dev(inst)
    Fg = dd.dd_nodal_forces(x, sn, b, n, SIG, MAT, Q)
    assert dd.dd_last_plan()[:2] == (inst.n_segs, inst.n_nodes)
    f, vel = torch.empty_like(x), torch.empty_like(x)
    dd.dd_step(x, sn, b, n, p, SIG, MAT, W.DT, Q, dd.DD_FP64, force_out=f, vel_out=vel)
    e = [normwise(Fg.cpu().numpy(), F), normwise(vel.cpu().numpy(), v), normwise(x.cpu().numpy() - inst.x, xn - inst.x)]
    print(f"{n_segs} segments, hub of {hub}, Q={Q}: forces {e[0]:.1e}, velocities {e[1]:.1e}, displacement {e[2]:.1e}")
    assert torch.equal(f, Fg)
    assert max(e[:2]) < 1e-10 and e[2] < 1e-9


@pytest.mark.parametrize("steps", [1, 2, 3, 4, 25])
def test_burst_vs_step_graph(steps):
    """Instances of 1 to 510 segments in one call (several nodes to a workgroup
    in the larger ones), against the step graph."""
    bt = W.pack([_network(20 + k, n, h) for k, (n, h) in enumerate([(1, 0), (64, 20), (130, 2), (510, 0), (33, 33)])])
    out = []
    for mode in (dd.BURST_AUTO, dd.BURST_GRAPH):
        prev = dd.dd_set_burst_mode(mode)
        try:
            x, sn, b, n, p = _dev(bt)
            sig, vol = (torch.tensor(a, device="cuda:0") for a in (bt.sigma_app, bt.volume))
            r, f = dd.dd_burst_batch(bt.node_off, bt.seg_off, x, sn, b, n, p, sig, vol, MAT, 2, dd.DD_FP64, 20.0, steps,
                                     W.DT / 10, want_features=True)
            out.append([a.cpu().numpy() for a in (x, r, f)])
        finally:
            dd.dd_set_burst_mode(prev)
    (xa, ra, fa), (xg, rg, fg) = out
    e = normwise(xa - bt.x, xg - bt.x)
    print(f"{steps} steps: displacement {e:.1e}, rates {np.abs(ra - rg).max() / np.abs(rg).max():.1e}")
    assert e < 1e-10
    assert np.abs(ra - rg).max() < 1e-12 * np.abs(rg).max()
    np.testing.assert_array_equal(fa, fg)


@pytest.mark.parametrize("n", [1, 2, 255, 256, 257])
def test_step_moves_every_node_once(n):
    """The nodes are moved by the last workgroup of the launch (up to 256 nodes)
    or by a launch of their own: every step moves every node by its velocity
    times dt, call after call (the count of the workgroups starts over), to the
    rounding of the two operations."""
    rng = np.random.default_rng(n)
    x0 = rng.uniform(0.0, 2000.0, (3, n))
    m = n if n > 2 else n - 1
    seg = np.stack([np.arange(m), (np.arange(m) + 1) % n]).astype(np.int32)
    b = rng.normal(size=(3, m))
    nrm = np.repeat(np.array([[0.0], [0.0], [1.0]]), m, axis=1)
    t = [torch.tensor(np.ascontiguousarray(a), device="cuda:0") for a in (seg, b / np.linalg.norm(b, axis=0), nrm)]
    x = torch.tensor(x0, device="cuda:0")
    vel = torch.empty_like(x)
    sig = np.array([1e7, -2e7, 5e7, 3e6, -4e6, 2e7])
    step = lambda: dd.dd_step(x, *t, None, sig, MAT, W.DT, n_gauss=2, vel_out=vel)   # noqa: E731
    for k in range(4):
        before = x.clone()
        step()
        np.testing.assert_allclose(x.cpu().numpy(), (before + vel * W.DT).cpu().numpy(), rtol=1e-15, atol=0)
        assert m == 0 or not torch.equal(x, before)
