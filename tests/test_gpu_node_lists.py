"""Node lists (node -> attached segment ends) at the sizes where their
construction changes: one workgroup per instance up to 16 K words (nodes + 2
segments), then separate launches.  The lists are seen through
dd_glide_step (length and slip planes of a node's segments), with nodes that no
segment uses and a hub with long lists.  Against the oracle, 1e-10 normwise (the
library's FP64 bound; the arithmetic is a handful of operations per node).
"""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2005_02498_amd as dd
from gpu_util import MAT, normwise
from paper_2005_02498_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nodes,segs,hub", [(2, 1, 0), (5, 3, 2), (65, 64, 40), (1000, 1107, 300), (5462, 5461, 20),
                                            (5463, 5461, 20), (12971, 12971, 9), (64, 20000, 0)])
def test_lists_through_glide(nodes, segs, hub):
    rng = np.random.default_rng(nodes)
    x = rng.uniform(0.0, 3000.0, (3, nodes))
    # each segment between two different nodes, the first `hub` of them at node 0;
    # one slip plane per node pair parity, so that nodes see one to three planes
    a = rng.integers(0, max(nodes - 1, 1), segs)
    b = (a + rng.integers(1, nodes, segs)) % nodes
    a[:hub] = 0
    b[:hub] = rng.integers(1, nodes, hub)
    seg = np.ascontiguousarray(np.stack([a, b]).astype(np.int32))
    planes = np.array([[1, 1, 1], [1, 1, -1]]) / np.sqrt(3.0)
    normal = np.ascontiguousarray(planes[(rng.random(segs) < 0.1).astype(int)].T)
    pinned = (rng.random(nodes) < 0.1).astype(np.uint8)
    F = rng.normal(size=(3, nodes)) * 1e-6
    xd = torch.tensor(x, device="cuda:0")
    v = dd.dd_glide_step(xd, torch.tensor(F, device="cuda:0"), torch.tensor(seg, device="cuda:0"),
                         torch.tensor(normal, device="cuda:0"), torch.tensor(pinned, device="cuda:0"), MAT, W.DT)
    xo, vo = O.glide_step(x.copy(), F, seg, normal, pinned, W.DRAG_B, W.DT)
    assert np.linalg.norm(vo) > 0.0 or nodes < 10
    e_v = normwise(v.cpu().numpy(), vo) if np.linalg.norm(vo) > 0.0 else np.abs(v.cpu().numpy()).max()
    e_x = normwise(xd.cpu().numpy(), xo)
    print(f"{nodes} nodes, {segs} segments: v {e_v:.2e}, x {e_x:.2e}")
    assert e_v < 1e-10 and e_x < 1e-10


def test_bad_segments_leave_the_other_nodes_alone():
    """A segment with an index out of range is attached to nothing; with
    validation off the call returns, the rest of the volume moves as if it were
    not there, and the flag is reported later."""
    rng = np.random.default_rng(3)
    n = 200
    x = rng.uniform(0.0, 3000.0, (3, n))
    seg = np.stack([np.arange(n), (np.arange(n) + 1) % n]).astype(np.int32)
    normal = np.ascontiguousarray(np.repeat(np.array([[0.0], [0.0], [1.0]]), n, axis=1))
    F = rng.normal(size=(3, n)) * 1e-6
    bad = seg.copy()
    bad[0, 17], bad[1, 60], bad[1, n - 1] = -1, n, 1 << 30
    keep = np.setdiff1d(np.arange(n), [17, 60, n - 1])
    old = dd.dd_set_validation(0)
    try:
        xd = torch.tensor(x, device="cuda:0")
        v = dd.dd_glide_step(xd, torch.tensor(F, device="cuda:0"), torch.tensor(bad, device="cuda:0"),
                             torch.tensor(normal, device="cuda:0"), None, MAT, W.DT)
        torch.cuda.synchronize()
    finally:
        dd.dd_set_validation(old)
    _, vo = O.glide_step(x.copy(), F, np.ascontiguousarray(seg[:, keep]), np.ascontiguousarray(normal[:, keep]),
                         np.zeros(n, np.uint8), W.DRAG_B, W.DT)
    assert normwise(v.cpu().numpy(), vo) < 1e-10
