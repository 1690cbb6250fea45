"""GPU parity of the all-pairs kernels on runs of sources that share a Burgers
vector, at every length around the one where the run form takes over: chains
cut into stretches of 1, 2, 3, ... segments that each carry their own random
Burgers vector, so that runs also end inside a chain, at work-item borders and
at the tile's own segments.

Tolerances: the library's stated bounds against the FP64 oracle, 1e-10 (FP64)
and 1e-4 (mixed), normwise.
"""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2005_02498_amd as dd
from gpu_util import MAT, normwise
from paper_2005_02498_amd import workloads as W

pytestmark = pytest.mark.gpu


def _chains(seed, stretches):
    """One closed polygon per stretch list entry (its segments share one
    Burgers vector), then one polygon whose Burgers vector changes after 1, 2,
    3, ... segments."""
    rng = np.random.default_rng(seed)
    xs, segs, bs, nrm, n0 = [], [], [], [], 0

    def polygon(lengths):
        nonlocal n0
        n = sum(lengths)
        c = rng.uniform(0.0, 1500.0, 3)
        u, v = np.linalg.qr(rng.normal(size=(3, 2)))[0].T
        ang = 2.0 * np.pi * (np.arange(n) + rng.uniform(0.0, 0.2, n)) / n
        xs.append(c[:, None] + 150.0 * (u[:, None] * np.cos(ang) + v[:, None] * np.sin(ang)))
        segs.append(np.stack([n0 + np.arange(n), n0 + (np.arange(n) + 1) % n]))
        for m in lengths:
            b = rng.normal(size=3)
            bs.append(np.repeat((b / np.linalg.norm(b))[:, None], m, axis=1))
        w = np.cross(u, v)
        nrm.append(np.repeat(w[:, None], n, axis=1))
        n0 += n

    for m in stretches:
        polygon([max(m, 3)])
        polygon([m] * (6 if m > 2 else 9))
    polygon(list(range(1, 14)))
    x = np.ascontiguousarray(np.concatenate(xs, axis=1))
    return W.Instance(x, np.ascontiguousarray(np.concatenate(segs, axis=1).astype(np.int32)),
                      np.ascontiguousarray(np.concatenate(bs, axis=1)),
                      np.ascontiguousarray(np.concatenate(nrm, axis=1)), np.zeros(x.shape[1], np.uint8),
                      np.array([1e7, -2e7, 5e7, 3e6, -4e6, 2e7]), 1e9)


@pytest.mark.parametrize("Q,chunk,variant", [(1, 0, 0), (2, 16, 2), (3, 32, 0), (4, 80, 2), (2, 512, 1)])
def test_short_runs_vs_oracle(Q, chunk, variant):
    inst = _chains(11, [1, 2, 3, 4, 5, 6, 7, 8, 9, 17, 33])
    ref = O.nodal_forces(inst.x, inst.seg_nodes, inst.burgers, inst.sigma_app, W.MU, W.NU, W.CORE_A, Q)
    dev = torch.device("cuda:0")
    args = [torch.tensor(a, device=dev) for a in (inst.x, inst.seg_nodes, inst.burgers, inst.normal)]
    dd.dd_set_plan(chunk, variant)
    try:
        for prec, tol in ((dd.DD_FP64, 1e-10), (dd.DD_MIXED, 1e-4)):
            F = dd.dd_nodal_forces(*args, inst.sigma_app, MAT, Q, prec, 20.0).cpu().numpy()
            e = normwise(F, ref)
            print(f"runs: {inst.n_segs} segments Q={Q} chunk={chunk} variant={variant} precision={prec} err {e:.2e}")
            assert e < tol
    finally:
        dd.dd_set_plan(-1)


@pytest.mark.parametrize("nseg", [27, 32])
@pytest.mark.parametrize("Q,variant", [(2, 0), (2, 2), (4, 2), (3, 0)])
def test_mixed_safe_sources_vs_oracle(nseg, Q, variant):
    """The mixed kernel's loop without tests: loops of 32 segments (each
    wavefront's target points share a Burgers vector at 2 and 4 points) and of
    27 (they do not), a source range that is no multiple of 64; every pair it
    takes by quadrature is counted as such."""
    rng = np.random.default_rng(3)
    x, seg, bur, nrm, _ = W._loops(rng, 19, 9000.0, 100.0, 500.0, nseg=nseg)
    sig = W.uniaxial_001(50e6)
    ref = O.nodal_forces(x, seg, bur, sig, W.MU, W.NU, W.CORE_A, Q)
    dev = torch.device("cuda:0")
    args = [torch.tensor(a, device=dev) for a in (x, seg, bur, nrm)]
    dd.dd_set_plan(200, variant)
    try:
        dd.dd_timing_read(reset=True)
        F = dd.dd_nodal_forces(*args, sig, MAT, Q, dd.DD_MIXED, 20.0).cpu().numpy()
        quad = dd.dd_timing_read(reset=True)[3]
    finally:
        dd.dd_set_plan(-1)
    e = normwise(F, ref)
    share = quad / (Q * (19.0 * nseg) ** 2)
    print(f"mixed {nseg} segments a loop Q={Q} variant={variant}: err {e:.2e}, quadrature share {share:.2f}")
    assert e < 1e-4
    assert share > 0.5
