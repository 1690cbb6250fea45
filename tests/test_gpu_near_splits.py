"""GPU parity of the exact band where the near search cuts the source groups
into splits: volumes of one group, of one split more or less, of a last split
that is short or empty, with the segments in no order (every group's sphere is
wide), and a batch whose small volumes leave most splits without a source.

Tolerance: the FP64 path's stated bound against the oracle, 1e-10, normwise.
"""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2005_02498_amd as dd
from gpu_util import MAT, batch_dev, normwise
from paper_2005_02498_amd import workloads as W

pytestmark = pytest.mark.gpu

ETA = 2.0


@pytest.fixture(autouse=True)
def _oracle_band():
    O.set_exact_band(ETA)
    yield
    O.set_exact_band(0.0)


@pytest.mark.parametrize("n", [7, 8, 63, 64, 65, 127, 129, 513, 1107])
def test_ragged_shuffled_volumes(n):
    inst = W.subset(W.config1(), 36)
    keep = np.random.default_rng(n).permutation(inst.seg_nodes.shape[1])[:n]
    seg = np.ascontiguousarray(inst.seg_nodes[:, keep])
    bur, nrm = np.ascontiguousarray(inst.burgers[:, keep]), np.ascontiguousarray(inst.normal[:, keep])
    x = inst.x * 0.25   # dense enough that shuffled segments have near ones
    t = [torch.tensor(a, device="cuda:0") for a in (x, seg, bur, nrm)]
    F = dd.dd_nodal_forces(*t, inst.sigma_app, MAT, 2, dd.DD_FP64, exact_eta=ETA).cpu().numpy()
    ref = O.nodal_forces(x, seg, bur, inst.sigma_app, W.MU, W.NU, W.CORE_A, 2)
    e = normwise(F, ref)
    print(f"{n} segments: err {e:.2e}")
    assert e < 1e-10


def test_uneven_batch():
    insts = [W.subset(W.config1(), nl) for nl in (1, 20, 2)]
    bt = W.pack(insts)
    d = batch_dev(bt)
    rate, _ = dd.dd_burst_batch(bt.node_off, bt.seg_off, d["x"], d["seg_nodes"], d["burgers"], d["normal"],
                                d["pinned"], d["sigma_app"], d["volume"], MAT, 2, dd.DD_FP64, 20.0, 1, W.DT,
                                exact_eta=ETA)
    torch.cuda.synchronize()
    xo, ro, _ = O.burst_batch(bt, W.material(), 2, 1, W.DT)
    assert normwise(d["x"].cpu().numpy() - bt.x, xo - bt.x) < 1e-10
    assert np.abs(rate.cpu().numpy() - ro).max() < 1e-10 * np.abs(ro).max()
