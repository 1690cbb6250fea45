"""What the work-split candidates of the autotuner leave in the workspace: the
partial sums of the shortest source range that a volume of its size is offered,
64 sources from about two thousand segments on, with the workspace's quarter of
headroom.  Shorter ranges would take twice that and more."""
import numpy as np
import pytest
import torch

import paper_2005_02498_amd as dd
from gpu_util import MAT
from paper_2005_02498_amd import workloads as W

pytestmark = pytest.mark.gpu

TILE = 256


def test_memory_of_a_tuned_call():
    # 7 points: a class of problems that no other test tunes
    Q, loops = 7, 400
    x, seg, bur, nrm, _ = W._loops(np.random.default_rng(5), loops, 20000.0, 100.0, 500.0)
    t = [torch.tensor(np.ascontiguousarray(a), device="cuda:0") for a in (x, seg.astype(np.int32), bur, nrm)]
    n = seg.shape[1]
    F = torch.empty_like(t[0])
    items = -(-n * Q // TILE) * -(-n // 64)
    sums = items * 3 * TILE * 8
    rest = n * 8 * (16 + 16 + 6) + (items + 1024) * 32   # records, end forces, plan
    assert sums > 400 << 20
    # the library's first use, which brings its fixed 64 MiB array (dd.h) to the device
    dd.dd_nodal_forces(t[0], *(a[:, :32].contiguous() for a in t[1:]), W.uniaxial_001(50e6), MAT, Q, dd.DD_FP64,
                       force_out=F)
    dd.dd_shutdown()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    free = torch.cuda.mem_get_info()[0]
    dd.dd_nodal_forces(*t, W.uniaxial_001(50e6), MAT, Q, dd.DD_FP64, force_out=F)
    torch.cuda.synchronize()
    used = free - torch.cuda.mem_get_info()[0]
    print(f"{n} segments, Q={Q}: {used / 2**20:.0f} MiB held, partial sums of ranges of 64 {sums / 2**20:.0f} MiB")
    assert used < 1.25 * (sums + rest) + (64 << 20)


def test_shortest_range_stays_with_the_small_volumes():
    """Volumes of 1,536 and 2,048 segments are of one class by size; ranges of 32,
    offered to the first, are not taken over for the second, which has work items
    enough without them."""
    for loops in (48, 64):
        x, seg, bur, nrm, _ = W._loops(np.random.default_rng(loops), loops, 8000.0, 100.0, 500.0)
        t = [torch.tensor(np.ascontiguousarray(a), device="cuda:0") for a in (x, seg.astype(np.int32), bur, nrm)]
        dd.dd_nodal_forces(*t, W.uniaxial_001(50e6), MAT, 2, dd.DD_FP64)
        print(seg.shape[1], dd.dd_last_plan())
    assert seg.shape[1] == 2048 and dd.dd_last_plan()[0] != 32
