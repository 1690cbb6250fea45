"""A node at infinity in a small FP64 volume: the one-launch step and the
persistent burst against the general kernels, whose velocities and positions are
NaN wherever the forces are (the segments at the node have infinite length, and
1 / (B ell) = 0 times a NaN force is no velocity of 0).  With validation on the call
is refused in either route.
"""
import numpy as np
import pytest
import torch

import paper_2005_02498_amd as dd
from gpu_util import MAT
from paper_2005_02498_amd import workloads as W

pytestmark = pytest.mark.gpu


def _volume(node):
    inst = W.config0()
    x = inst.x.copy()
    x[1, node] = np.inf
    return [torch.tensor(np.ascontiguousarray(a), device="cuda:0") for a in (x, inst.seg_nodes, inst.burgers, inst.normal)]


def _step(vol, general):
    x, f, v = vol[0].clone(), torch.zeros_like(vol[0]), torch.zeros_like(vol[0])
    if general:
        dd.dd_set_plan(64, 0)
    try:
        dd.dd_step(x, *vol[1:], None, W.uniaxial_001(50e6), MAT, 2e-16, 2, dd.DD_FP64, 20.0, force_out=f, vel_out=v)
    finally:
        dd.dd_set_plan(-1)
    return [a.cpu().numpy() for a in (x, f, v)]


def _burst(vol, mode, steps):
    x = vol[0].clone()
    nn, ns = x.shape[1], vol[1].shape[1]
    dev = x.device
    prev = dd.dd_set_burst_mode(mode)
    try:
        r, _ = dd.dd_burst_batch([0, nn], [0, ns], x, *vol[1:], None,
                                 torch.tensor(W.uniaxial_001(50e6)[None], device=dev),
                                 torch.tensor([8.0e9], dtype=torch.float64, device=dev), MAT, 2, dd.DD_FP64, 20.0,
                                 steps, 2e-16)
    finally:
        dd.dd_set_burst_mode(prev)
    return [a.cpu().numpy() for a in (x, r)]


@pytest.mark.parametrize("node", [0, 17, 255])
def test_infinite_position(node):
    vol = _volume(node)
    on = dd.dd_set_validation(False)
    try:
        small, general = _step(vol, False), _step(vol, True)
        for s, g, what in zip(small, general, ("positions", "forces", "velocities")):
            assert np.array_equal(np.isnan(s), np.isnan(g)), what
            assert np.isnan(g).any(), what
        for steps in (1, 3):
            for s, g in zip(_burst(vol, dd.BURST_AUTO, steps), _burst(vol, dd.BURST_GRAPH, steps)):
                assert np.array_equal(np.isnan(s), np.isnan(g)), steps
        with pytest.raises(dd.DDError):
            dd.dd_check()
        dd.dd_set_validation(True)
        for general in (False, True):
            with pytest.raises(dd.DDError):
                _step(vol, general)
    finally:
        dd.dd_set_validation(on)
