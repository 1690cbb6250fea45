"""A persistent burst whose workgroups wait too long for a position fails as a
whole.  The longest wait is set to nothing: a workgroup that finds a position
missing leaves the launch, and the others after it (256 workgroups that start one
after the other do not find every position there at their first look).  The
caller's positions stay as they were bit for bit, the rates are NaN, nothing of
an earlier burst shows, and the next burst is as before."""
import numpy as np
import pytest
import torch

import paper_2005_02498_amd as dd
from gpu_util import MAT, batch_dev
from paper_2005_02498_amd import workloads as W

pytestmark = pytest.mark.gpu


def _burst(d, bt, steps):
    return dd.dd_burst_batch(bt.node_off, bt.seg_off, d["x"], d["seg_nodes"], d["burgers"], d["normal"], d["pinned"],
                             d["sigma_app"], d["volume"], MAT, 2, dd.DD_FP64, 20.0, steps, W.DT)[0]


@pytest.mark.parametrize("validate", [True, False])
def test_a_burst_given_up_leaves_no_results(validate):
    bt = W.pack([W.subset(W.burst_instance(1_000_040 + i), nl) for i, nl in enumerate((3, 1, 8))])
    good = batch_dev(bt)
    ref = _burst(good, bt, 6).cpu()   # (and an earlier burst's results in the workspace)
    assert not torch.equal(good["x"].cpu(), torch.tensor(bt.x))
    d = batch_dev(bt)
    old_val = dd.dd_set_validation(validate)
    old_wait = dd.dd_set_burst_wait(0)
    try:
        if validate:
            with pytest.raises(dd.DDError, match="waited too long for a position"):
                _burst(d, bt, 6)
            d["rate"] = None
        else:
            d["rate"] = _burst(d, bt, 6)
            with pytest.raises(dd.DDError, match="waited too long for a position"):
                dd.dd_check()
        # one step needs no other workgroup's positions
        one = batch_dev(bt)
        assert torch.isfinite(_burst(one, bt, 1)).all()
    finally:
        dd.dd_set_burst_wait(old_wait)
        dd.dd_set_validation(old_val)
    np.testing.assert_array_equal(d["x"].cpu().numpy(), bt.x)
    if d["rate"] is not None:
        assert torch.isnan(d["rate"]).all()
    again = batch_dev(bt)
    assert torch.equal(_burst(again, bt, 6).cpu(), ref)
    assert torch.equal(again["x"], good["x"])


def test_wait_is_checked_and_returned():
    old = dd.dd_set_burst_wait(1234)
    assert dd.dd_set_burst_wait(old) == 1234
    for bad in (-1, 1 << 62):
        with pytest.raises(dd.DDError):
            dd.dd_set_burst_wait(bad)
    assert dd.dd_set_burst_wait(old) == old
