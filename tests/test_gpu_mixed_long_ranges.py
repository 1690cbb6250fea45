"""The mixed all-pairs kernel for long source ranges (512 sources and more),
which runs sources that every target point of a wavefront takes by quadrature
in a loop without tests, against the kernel for shorter ranges, which tests
every source.

Both flush FP32 sums to FP64 at the same 256 sources where ranges are multiples
of 256, and take every pair by the same arithmetic, so that the forces differ by
the order of FP64 sums alone: 1e-13 of the largest (FP32 differences are of the
order of 1e-8).  Ranges that end inside a stage or a group of 64 are compared
with the oracle, at the library's 1e-4.  Near-field and quadrature evaluations
are counted alike to the last one.
"""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2005_02498_amd as dd
from gpu_util import MAT, normwise
from paper_2005_02498_amd import workloads as W

pytestmark = pytest.mark.gpu


def _volume(loops, nseg, box, shuffle=False):
    rng = np.random.default_rng(loops + nseg)
    x, seg, bur, nrm, _ = W._loops(rng, loops, box, 100.0, 500.0, nseg=nseg)
    if shuffle:   # all segments, or the first half: targets scattered in every work item, or in some
        m = seg.shape[1] if shuffle == "all" else seg.shape[1] // 2
        p = np.concatenate([rng.permutation(m), np.arange(m, seg.shape[1])])
        seg, bur, nrm = seg[:, p], bur[:, p], nrm[:, p]
    return x, seg.astype(np.int32), bur, nrm


def _forces(vol, Q, chunk, variant):
    t = [torch.tensor(np.ascontiguousarray(a), device="cuda:0") for a in vol]
    dd.dd_set_plan(chunk, variant)
    try:
        dd.dd_timing_read(reset=True)
        F = dd.dd_nodal_forces(*t, W.uniaxial_001(50e6), MAT, Q, dd.DD_MIXED, 20.0).cpu().numpy()
        _, _, near, quad = dd.dd_timing_read(reset=True)
        assert dd.dd_last_plan()[0] == chunk and dd.dd_last_plan()[2] == variant
    finally:
        dd.dd_set_plan(-1)
    return F, near, quad


# loops of 32 segments: a wavefront's target points share their Burgers vector
# at 2 points (one loop) and 4 (half of one); of 27, or at 3 points, or shuffled:
# most do not.  Volumes of 640 to 1,188 segments: stages of 256 with tails of
# 128, 130, 164 and 47.  The densest volume leaves much to the tests.
@pytest.mark.parametrize("loops,nseg,box,shuffle,Q", [
    (20, 32, 9000.0, False, 2), (20, 32, 9000.0, False, 4), (33, 27, 9000.0, False, 2), (36, 33, 9000.0, False, 3),
    (20, 32, 9000.0, "all", 2), (48, 32, 9000.0, "half", 2), (24, 32, 1500.0, False, 2),
    (49, 16, 9000.0, False, 1), (815, 1, 9000.0, False, 2)])
@pytest.mark.parametrize("variant", [0, 2])
def test_same_as_with_short_ranges(loops, nseg, box, shuffle, Q, variant):
    if nseg == 1:   # separate straight segments, no two with one Burgers vector
        rng = np.random.default_rng(0)
        a = rng.uniform(0.0, box, (3, loops))
        vol = (np.concatenate([a, a + rng.normal(size=a.shape) * 40.0], axis=1),
               np.stack([np.arange(loops), loops + np.arange(loops)]).astype(np.int32), rng.normal(size=a.shape),
               np.repeat(np.array([[0.0], [0.0], [1.0]]), loops, axis=1))
    else:
        vol = _volume(loops, nseg, box, shuffle)
    short = _forces(vol, Q, 256, variant)
    for chunk in (512, 1024, 4096):
        long = _forces(vol, Q, chunk, variant)
        d = np.abs(long[0] - short[0]).max() / np.abs(short[0]).max()
        print(f"{vol[1].shape[1]} segments Q={Q} variant={variant} range {chunk}: {d:.1e}, near {long[1]}, quad {long[2]}")
        assert d < 1e-13
        assert long[1:] == short[1:]
    assert short[2] > 0


@pytest.mark.parametrize("chunk", [512, 520, 700, 961])
@pytest.mark.parametrize("nseg,Q,variant", [(27, 2, 0), (27, 4, 2), (32, 2, 2), (32, 4, 0), (31, 3, 2), (31, 1, 0)])
def test_ragged_ranges_vs_oracle(nseg, Q, variant, chunk):
    vol = _volume(1100 // nseg, nseg, 9000.0)
    assert vol[1].shape[1] > chunk
    ref = O.nodal_forces(*vol[:3], W.uniaxial_001(50e6), W.MU, W.NU, W.CORE_A, Q)
    F, near, quad = _forces(vol, Q, chunk, variant)
    exact = _forces(vol, Q, chunk, 1)[0]   # every pair located in FP64
    e = normwise(F, ref)
    share = quad / (Q * float(vol[1].shape[1]) ** 2)
    print(f"{vol[1].shape[1]} segments Q={Q} variant={variant} range {chunk}: err {e:.2e} (variant 1 "
          f"{normwise(exact, ref):.2e}), quadrature share {share:.2f}")
    assert e < 1e-4
    assert share > 0.3
