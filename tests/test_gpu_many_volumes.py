"""Junction-node bursts of more volumes than get a workgroup each for their node
lists (four per compute unit): the same volumes' results from smaller batches,
whose lists are built that way, are the same - topology, junction state and
counts bit for bit, positions and rates to the rounding of another work split
(1e-12)."""
import numpy as np
import pytest
import torch

import paper_2005_02498_amd as dd
from gpu_util import MAT
from paper_2005_02498_amd import workloads as W

pytestmark = pytest.mark.gpu

K = 2


def _run(insts, frac, calls):
    bt = W.pack(insts)
    x, sn, bu, nr, pin, sig, vol = (torch.tensor(a, device="cuda:0") for a in (
        bt.x, bt.seg_nodes, bt.burgers, bt.normal, bt.pinned, bt.sigma_app, bt.volume))
    st = dd.junction_node_state(int(bt.node_off[-1]), int(bt.seg_off[-1]), bt.n_inst, torch.device("cuda:0"))
    rates = [dd.dd_burst_batch_junction_nodes(bt.node_off, bt.seg_off, x, sn, bu, nr, pin, sig, vol, MAT, st,
                                              torch.tensor(frac, device="cuda:0"), 30.0, 6.0 * W.DT, 1.0, K,
                                              t0=c * 5 * W.DT, n_gauss=2, precision=dd.DD_FP64, n_steps=5,
                                              dt=W.DT)[0].clone() for c in range(calls)]
    off = torch.repeat_interleave(torch.tensor(bt.seg_off[:-1]), torch.tensor(np.diff(bt.node_off))).cuda()
    st["ses"] = torch.where(st["ses"] >= 0, st["ses"] - off.to(torch.int32), st["ses"])   # (within the volume)
    return bt, [a.cpu().numpy() for a in (sn, bu, st["ses"], st["ignore"], st["count"], st["missed"], x)], rates


def test_more_volumes_than_list_workgroups():
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    kinds = []
    for k in range(3):   # a mobile loop of 8 or 12 segments beside pinned ones
        x, seg, bur, nrm, _ = W._loops(np.random.default_rng(70 + k), 3, 300.0, 60.0, 120.0, nseg=8 + 4 * (k % 2))
        pin = np.ones(x.shape[1], np.uint8)
        pin[:seg.shape[1] // 3] = 0
        kinds.append(W.with_junction_slots(W.Instance(x, seg.astype(np.int32), bur, nrm, pin, W.uniaxial_001(2e8), 1e7), K))
    n = 4 * cus + 1
    frac = np.random.default_rng(1).uniform(0.1, 1.0, (3, 4))
    bt, big, rb = _run([kinds[i % 3] for i in range(n)], frac[np.arange(n) % 3], 3)
    st, small, rs = _run(kinds, frac, 3)
    assert small[4].sum() > 0   # junctions formed
    for i in (0, 1, 2, n // 2, n - 2, n - 1):
        k = i % 3
        nb, sb = slice(*bt.node_off[i:i + 2]), slice(*bt.seg_off[i:i + 2])
        ns, ss = slice(*st.node_off[k:k + 2]), slice(*st.seg_off[k:k + 2])
        for a, b, p, q in ((big[0], small[0], sb, ss), (big[1], small[1], sb, ss)):
            np.testing.assert_array_equal(a[:, p], b[:, q])
        np.testing.assert_array_equal(big[2][nb], small[2][ns])
        np.testing.assert_array_equal(big[3][sb], small[3][ss])
        assert big[4][i] == small[4][k] and big[5][i] == small[5][k]
        assert np.abs(big[6][:, nb] - small[6][:, ns]).max() < 1e-12 * np.abs(small[6][:, ns]).max()
        for a, b in zip(rb, rs):
            a, b = a.cpu().numpy(), b.cpu().numpy()
            assert np.abs(a[i] - b[k]).max() <= 1e-12 * np.abs(b).max()
