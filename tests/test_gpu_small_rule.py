"""Which single FP64 volumes take the one launch of small volumes: those with at
most three rounds of target points for a workgroup of mean valence, one beyond 8
points (a workgroup takes every segment of its node: a round is 16, 8, 4 or 2 points for up to 64,
128, 256 or 512 segments).  On both sides of the line, with a node of many
segments too, against the FP64 oracle at the library's 1e-10."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2005_02498_amd as dd
from gpu_util import MAT, normwise
from paper_2005_02498_amd import workloads as W

pytestmark = pytest.mark.gpu


def _volume(segs, nodes, hub):
    """A closed chain through all nodes, more segments between nodes at random,
    the last `hub` of them at node 0."""
    rng = np.random.default_rng(segs + nodes)
    x = rng.uniform(0.0, 2000.0, (3, nodes))
    a = np.arange(segs) % nodes
    b = (a + 1) % nodes
    extra = np.arange(segs) >= nodes
    b[extra] = (a[extra] + rng.integers(2, max(nodes - 1, 3), extra.sum())) % nodes
    if hub:
        a[-hub:], b[-hub:] = 0, 2 + rng.choice(nodes - 2, hub, replace=False)
    bur = rng.normal(size=(3, segs))
    nrm = np.repeat(np.array([[0.0], [0.0], [1.0]]), segs, axis=1)
    return x, np.ascontiguousarray(np.stack([a, b]).astype(np.int32)), bur / np.linalg.norm(bur, axis=0), nrm


@pytest.mark.parametrize("segs,nodes,hub,Q,small", [
    (256, 256, 0, 6, True), (256, 256, 0, 7, False), (256, 256, 0, 8, False), (254, 254, 16, 8, False),
    (512, 512, 0, 3, True), (512, 512, 0, 4, False), (496, 496, 16, 4, False), (496, 496, 16, 16, False),
    (128, 128, 0, 8, True), (128, 128, 0, 9, False), (64, 64, 0, 8, True), (64, 64, 16, 16, False),
    (32, 64, 0, 16, True), (500, 60, 0, 1, False),
    (257, 257, 0, 3, True), (257, 257, 0, 4, False), (64, 8, 0, 3, True), (64, 8, 0, 4, False)])
def test_route_and_forces(segs, nodes, hub, Q, small):
    x, seg, bur, nrm = _volume(segs, nodes, hub)
    sig = np.array([2e7, -3e7, 5e7, 1e7, -2e7, 4e7])
    ref = O.nodal_forces(x, seg, bur, sig, W.MU, W.NU, W.CORE_A, Q)
    t = [torch.tensor(a, device="cuda:0") for a in (x, seg, bur, nrm)]
    dd.dd_set_plan(-1)
    F = dd.dd_nodal_forces(*t, sig, MAT, Q, dd.DD_FP64)
    plan = dd.dd_last_plan()[:2]
    G = torch.empty_like(F)
    dd.dd_nodal_forces_noalloc(*t, sig, MAT, G, Q, dd.DD_FP64)
    e = normwise(F.cpu().numpy(), ref), normwise(G.cpu().numpy(), ref)
    print(f"{segs} segments, {nodes} nodes, node of {hub}, Q={Q}: plan {plan}, err {e[0]:.1e} {e[1]:.1e}")
    assert (plan == (segs, nodes)) == small
    assert max(e) < 1e-10
