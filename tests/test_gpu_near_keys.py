"""The exact band's keys and spheres come with the segment records where a
volume's node lists fit one workgroup, and in a launch of their own where they
do not: the same volume, made too large for the first by nodes that no segment
uses, has the same forces bit for bit (the search, the order of its pairs and
the sums are the same), at numbers of segments around a workgroup's share.
"""
import numpy as np
import pytest
import torch

import paper_2005_02498_amd as dd
from gpu_util import MAT
from paper_2005_02498_amd import workloads as W

pytestmark = pytest.mark.gpu

LISTS = 16 * 1024   # nodes + 2 segments of a volume whose lists one workgroup builds


@pytest.mark.parametrize("precision", [dd.DD_FP64, dd.DD_MIXED])
@pytest.mark.parametrize("n", [1, 8, 255, 256, 257, 1023, 1107])
def test_same_forces_as_with_a_launch_for_the_keys(n, precision):
    inst = W.subset(W.config1(), 36)
    keep = np.random.default_rng(n).permutation(inst.seg_nodes.shape[1])[:n]
    seg, bur, nrm = (np.ascontiguousarray(a[:, keep]) for a in (inst.seg_nodes, inst.burgers, inst.normal))
    x = inst.x * 0.25   # dense enough that shuffled segments have near ones
    nn = x.shape[1]
    assert nn + 2 * n <= LISTS
    xl = np.concatenate([x, np.zeros((3, LISTS + 1 - 2 * n - nn))], axis=1)
    t = [torch.tensor(a, device="cuda:0") for a in (seg, bur, nrm)]
    old = dd.dd_set_autotune(0)
    try:
        F = [dd.dd_nodal_forces(torch.tensor(a, device="cuda:0"), *t, inst.sigma_app, MAT, 2, precision,
                                exact_eta=2.0).cpu() for a in (x, xl)]
        # (small FP64 volumes without the band have a route of their own; with it they do not)
        far = dd.dd_nodal_forces(torch.tensor(xl, device="cuda:0"), *t, inst.sigma_app, MAT, 2, precision).cpu()
    finally:
        dd.dd_set_autotune(old)
    assert torch.equal(F[0], F[1][:, :nn])
    assert not F[1][:, nn:].any()
    if n >= 255:
        assert not torch.equal(F[1], far)   # the band has pairs
