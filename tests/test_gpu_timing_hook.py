"""Event timing measures and changes nothing: with it on, evaluations and steps
take the same route and return the same bits, and each all-pairs launch is
counted once, for volumes on both sides of the small-volume route."""
import pytest
import torch

import paper_2005_02498_amd as dd
from gpu_util import MAT, dev
from paper_2005_02498_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("loops", [1, 8, 16, 17, 40])
def test_timing_changes_nothing(loops):
    inst = W.subset(W.config1(), loops)
    out = []
    for on in (False, True):
        d = dev(inst)
        old = dd.dd_timing_enable(on)
        try:
            dd.dd_timing_read(reset=True)
            F = dd.dd_nodal_forces(d["x"], d["seg_nodes"], d["burgers"], d["normal"], inst.sigma_app, MAT, 2)
            plan = dd.dd_last_plan()
            f, v = torch.empty_like(F), torch.empty_like(F)
            dd.dd_step(d["x"], d["seg_nodes"], d["burgers"], d["normal"], d["pinned"], inst.sigma_app, MAT, W.DT, 2,
                       force_out=f, vel_out=v)
            ms, launches, _, _ = dd.dd_timing_read(reset=True)
        finally:
            dd.dd_timing_enable(old)
        out.append((F, f, v, d["x"], plan, launches, ms))
    (off, on) = out
    assert all(torch.equal(a, b) for a, b in zip(off[:4], on[:4]))
    assert off[4] == on[4]
    assert (off[5], on[5]) == (0, 2) and on[6] > 0.0
