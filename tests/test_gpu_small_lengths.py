"""Segment lengths and directions of the small-volume route are as accurate as
the general one's.  One segment of a volume by itself, one point: the force at
its nodes is half of (sigma b) x d, d the segment, to which the length L and the
direction d / L contribute only their rounding errors.  Over many segments the
root mean square error against extended precision is compared between the two
routes on the same inputs.

Both take sqrt and 1 / L, so the errors should be alike; a form with one more
rounding of the length and an inverse whose error counts twice has (by the
variance of its roundings) a mean square error half as large again, 1.2 times in
the root.  3 x 1,500 values leave 2 % of statistical error to a ratio: 1.1.
"""
import numpy as np
import torch
import pytest

import paper_2005_02498_amd as dd
from gpu_util import MAT
from paper_2005_02498_amd import workloads as W

pytestmark = pytest.mark.gpu


def test_rounding_of_a_single_segment():
    rng = np.random.default_rng(8)
    N = 1500
    d = rng.normal(size=(N, 3))
    d *= (10.0 ** rng.uniform(-3.0, 3.0, N) / np.linalg.norm(d, axis=1))[:, None]
    b = rng.normal(size=(N, 3))
    sig = np.array([2e7, -3e7, 5e7, 1e7, -2e7, 4e7])
    S = np.array([[sig[0], sig[5], sig[4]], [sig[5], sig[1], sig[3]], [sig[4], sig[3], sig[2]]])
    x = torch.tensor(np.stack([np.zeros((N, 3)), d], axis=2), device="cuda:0")   # node 0 in the origin
    bd = torch.tensor(b[:, :, None].copy(), device="cuda:0")
    seg = torch.tensor([[0], [1]], dtype=torch.int32, device="cuda:0")
    nrm = torch.tensor([[0.0], [0.0], [1.0]], dtype=torch.float64, device="cuda:0")
    dl, bl, Sl = d.astype(np.longdouble), b.astype(np.longdouble), S.astype(np.longdouble)
    ref = np.cross(bl @ Sl, dl) / 2
    err = []
    old = dd.dd_set_validation(False)
    try:
        for plan in (-1, 64):
            dd.dd_set_plan(plan)
            F = torch.stack([dd.dd_nodal_forces(x[i], seg, bd[i], nrm, sig, MAT, 1) for i in range(N)])
            assert (dd.dd_last_plan()[:2] == (1, 2)) == (plan < 0)
            e = (F[:, :, 0].cpu().numpy().astype(np.longdouble) - ref) / np.linalg.norm(ref, axis=1)[:, None]
            err.append(float(np.sqrt((e * e).mean())))
    finally:
        dd.dd_set_plan(-1)
        dd.dd_set_validation(old)
    print(f"rms error: small-volume route {err[0]:.3e}, general route {err[1]:.3e}")
    assert err[0] < 1.1 * err[1]
