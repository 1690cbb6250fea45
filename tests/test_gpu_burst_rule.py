"""Which batches of small FP64 bursts run in the persistent launch: those whose
workgroups, of as few nodes as there are compute units for, take at most 12
rounds of target points (a round is 16, 8, 4 or 2 points for up to 64, 128, 256
or 512 segments).  On both sides of the line, the launch against the step graph
at 1e-12, and the graph itself bit for bit where the line leaves it the call."""
import numpy as np
import pytest
import torch

import paper_2005_02498_amd as dd
from gpu_util import MAT, batch_dev
from paper_2005_02498_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("inst,loops,Q,rounds", [(1, 8, 2, 1), (16, 8, 2, 9), (8, 8, 4, 9), (12, 8, 4, 13), (24, 8, 2, 13),
                                                (1, 16, 8, 12), (2, 16, 8, 20), (64, 2, 8, 9), (64, 2, 12, 13)])
def test_route_of_a_batch(inst, loops, Q, rounds):
    bt = W.pack([W.subset(W.burst_instance(1_000_060 + i), loops) for i in range(inst)])
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    segs = 32 * loops
    if cus != 256:
        pytest.skip("the rounds are those of 256 compute units")
    npw = -(-inst * segs // cus)
    assert -(-(npw + 1) * Q // (512 // max(64, segs) * 2)) == rounds
    out = []
    for mode in (dd.BURST_AUTO, dd.BURST_GRAPH):
        d = batch_dev(bt)
        old = dd.dd_set_burst_mode(mode)
        try:
            r, _ = dd.dd_burst_batch(bt.node_off, bt.seg_off, d["x"], d["seg_nodes"], d["burgers"], d["normal"],
                                     d["pinned"], d["sigma_app"], d["volume"], MAT, Q, dd.DD_FP64, 20.0, 3, W.DT)
        finally:
            dd.dd_set_burst_mode(old)
        out.append((d["x"].cpu().numpy(), r.cpu().numpy(), dd.dd_last_plan()))
    (xa, ra, pa), (xg, rg, pg) = out
    print(f"{inst} x {segs} segments, Q={Q}, {rounds} rounds: auto {pa}, graph {pg}")
    if rounds <= 12:
        assert pa == (segs, inst * -(-segs // npw), 0)
        assert np.abs(xa - xg).max() < 1e-12 * np.abs(xg).max()
        assert np.abs(ra - rg).max() < 1e-12 * np.abs(rg).max()
    else:
        assert pa == pg
        np.testing.assert_array_equal(xa, xg)
        np.testing.assert_array_equal(ra, rg)
