"""dd_last_plan speaks of the most recent evaluation on every route: the
all-pairs kernels, a small volume's one launch and the persistent launch of a
burst."""
import pytest
import torch

import paper_2005_02498_amd as dd
from gpu_util import MAT, batch_dev, dev
from paper_2005_02498_amd import workloads as W

pytestmark = pytest.mark.gpu


def _forces(inst, precision):
    d = dev(inst)
    dd.dd_nodal_forces(d["x"], d["seg_nodes"], d["burgers"], d["normal"], inst.sigma_app, MAT, 2, precision)


def _burst(bt, mode):
    d = batch_dev(bt)
    old = dd.dd_set_burst_mode(mode)
    try:
        dd.dd_burst_batch(bt.node_off, bt.seg_off, d["x"], d["seg_nodes"], d["burgers"], d["normal"], d["pinned"],
                          d["sigma_app"], d["volume"], MAT, 2, dd.DD_FP64, 20.0, 2, W.DT)
    finally:
        dd.dd_set_burst_mode(old)


def test_last_plan_on_every_route():
    inst = W.config0()
    bt = W.pack([inst, W.subset(inst, 3)])
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    dd.dd_set_plan(64, 1)
    try:
        _forces(inst, dd.DD_MIXED)
        assert dd.dd_last_plan() == (64, 2 * 4, 1)   # 512 points in tiles of 256, 256 sources
        _burst(bt, dd.BURST_PERSISTENT_ONE)
        assert dd.dd_last_plan() == (256, 2, 0)
        _forces(inst, dd.DD_MIXED)
        _burst(bt, dd.BURST_AUTO)
        chunk, items, variant = dd.dd_last_plan()
        assert (chunk, variant) == (256, 0) and 2 < items <= cus
        _forces(inst, dd.DD_MIXED)
        _burst(bt, dd.BURST_GRAPH)
        assert dd.dd_last_plan()[0] == 64
    finally:
        dd.dd_set_plan(-1)
    _forces(inst, dd.DD_FP64)
    assert dd.dd_last_plan() == (256, 256, 0)
