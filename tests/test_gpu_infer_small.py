"""Surrogate inference for few points (tiles of 32, the ensemble reduced by the
last member's workgroup) against the same points inside a large batch (tiles
of 128, a launch of its own for the ensemble): a point's results do not depend
on the batch it is in, bit for bit.  Sizes: a single point, the edges of a tile,
and the largest batch of the small form for every number of members (one tile
of each member per compute unit) and one tile more.
"""
import numpy as np
import pytest
import torch

import paper_2005_02498_amd as dd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("members", [1, 2, 3, 4, 5, 8])
@pytest.mark.parametrize("log_dens", [False, True])
def test_small_batches_equal_large(members, log_dens):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    edge = 32 * (cus // members)
    mdl = dd.SurrogateModel(members, 11)
    rng = np.random.default_rng(members)
    mdl.set_scaling(rng.normal(size=36), rng.uniform(0.5, 2.0, 36), rng.normal(size=12), rng.uniform(0.5, 2.0, 12))
    if log_dens:
        mdl.set_log_densities(1.0e-2, 1.0e-6)
    big = 4 * edge + 77
    feat = torch.tensor(rng.normal(size=(big, 36)).astype(np.float32), device="cuda:0")
    ref = [t.cpu().numpy() for t in dd.dd_surrogate_rates(mdl, feat, 0.9)]
    for n in (1, 5, 31, 32, 33, 64, 100, 1000, edge - 31, edge - 1, edge, edge + 1, edge + 33):
        for first in (0, big - n - (big - n) % 4):
            for _ in range(2):   # the count of a tile's members starts over
                got = dd.dd_surrogate_rates(mdl, feat[first:first + n].clone(), 0.9)
                for a, b in zip(got, ref):
                    np.testing.assert_array_equal(a.cpu().numpy(), b[first:first + n])


def test_copies_after_a_step_equal_fresh_ones():
    """Training writes the bfloat16 weight copies itself; they are those that
    setting the same parameters makes: inference, and the next gradients, agree
    bit for bit."""
    rng = np.random.default_rng(5)
    feat = torch.tensor(rng.normal(size=(333, 36)).astype(np.float32), device="cuda:0")
    tgt = torch.tensor(rng.normal(size=(333, 12)).astype(np.float32), device="cuda:0")
    a, b = dd.SurrogateModel(3, 1), dd.SurrogateModel(3, 2)
    for _ in range(3):
        dd.dd_mlp_train_step(a, feat, tgt, 1e-2)
    for m in range(3):
        b.set_params(m, a.get_params(m))
    for x, y in zip(dd.dd_surrogate_rates(a, feat), dd.dd_surrogate_rates(b, feat)):
        np.testing.assert_array_equal(x.cpu().numpy(), y.cpu().numpy())
    for x, y in zip(dd.dd_mlp_gradients(a, feat, tgt), dd.dd_mlp_gradients(b, feat, tgt)):
        np.testing.assert_array_equal(x.cpu().numpy(), y.cpu().numpy())
