"""Records and node lists of one volume in one launch, whose workgroups are four
times as wide as their share of segments: the same volume, made too large for
that launch by nodes that no segment uses, has its records and lists from
launches of their own and the same forces bit for bit (the arithmetic and the
order of every sum are the same), at numbers of segments around a workgroup's
share.  (Keys and spheres of the exact band in the same launch: test_gpu_near_keys.)
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
@pytest.mark.parametrize("n", [1, 63, 255, 256, 257, 512, 1025])
def test_same_forces_as_with_launches_of_their_own(n, precision):
    inst = W.subset(W.config1(), 33)   # loops in order: runs end at a workgroup's last segment
    seg, bur, nrm = (np.ascontiguousarray(a[:, :n]) for a in (inst.seg_nodes, inst.burgers, inst.normal))
    x = inst.x
    nn = x.shape[1]
    assert nn + 2 * n <= LISTS
    xl = np.concatenate([x, np.zeros((3, LISTS + 1 - 2 * n - nn))], axis=1)
    t = [torch.tensor(a, device="cuda:0") for a in (seg, bur, nrm)]
    dd.dd_set_plan(128, 0)   # (small FP64 volumes have a route of their own without a fixed plan)
    try:
        F = [dd.dd_nodal_forces(torch.tensor(a, device="cuda:0"), *t, inst.sigma_app, MAT, 2, precision).cpu()
             for a in (x, xl)]
    finally:
        dd.dd_set_plan(-1)
    assert torch.equal(F[0], F[1][:, :nn])
    assert F[0].any() and not F[1][:, nn:].any()
