"""dd_block_to_gauss at the mesh sizes where its solver changes: nodes of a
component in LDS (up to 89 x 89, one workgroup per component), then separate
launches for the load vector and the two sweeps.  Every node against a dense
solve: the in-plane system is a product of two one-dimensional ones, so that
one line's inverse, applied to the rows and to the columns of the load vector,
solves it (numpy, float64).  With m = 1 the eight Gauss points of a block see
its four corner nodes and nothing else.

Tolerance: the systems' condition number is below 6 per direction (eigenvalues
between 2 and 6 over h / 6, halved end rows aside), a few hundred roundings per
line: 1e-12 normwise.
"""
import numpy as np
import pytest
import torch

import paper_2005_02498_amd as dd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,c", [(1, 1), (6, 9), (7, 2), (8, 16), (31, 3), (50, 9), (87, 4), (88, 9), (89, 9), (90, 3)])
def test_every_gauss_point(n, c):
    B = 1.7
    rng = np.random.default_rng(n * 17 + c)
    f = rng.normal(size=(n * n, c))
    N = n + 1
    K = np.diag(np.full(N, 4.0)) + np.diag(np.ones(n), 1) + np.diag(np.ones(n), -1)
    K[0, 0] = K[-1, -1] = 2.0
    inv = np.linalg.inv(K * (B / 6.0))
    load = np.zeros((N, N, c))
    g = f.reshape(n, n, c)
    for dy in (0, 1):
        for dx in (0, 1):
            load[dy:dy + n, dx:dx + n] += 0.25 * B * B * g
    nodal = np.einsum("ab,bjc->ajc", inv, np.einsum("ab,jbc->jac", inv, load))
    gp = np.array([-1.0, 1.0]) / np.sqrt(3.0)
    ref = np.zeros((n, n, 2, 2, 2, c))   # element row, element, z, y, x
    for iy, eta in enumerate(gp):
        for ix, xi in enumerate(gp):
            w = [(1 - xi) * (1 - eta), (1 + xi) * (1 - eta), (1 - xi) * (1 + eta), (1 + xi) * (1 + eta)]
            v = 0.25 * (w[0] * nodal[:-1, :-1] + w[1] * nodal[:-1, 1:] + w[2] * nodal[1:, :-1] + w[3] * nodal[1:, 1:])
            ref[:, :, :, iy, ix] = v[:, :, None]
    got = dd.dd_block_to_gauss(torch.tensor(f, device="cuda:0"), n, 1, B, 0.3).cpu().numpy()
    e = np.abs(got.reshape(ref.shape) - ref).max() / np.abs(ref).max()
    print(f"n={n} c={c}: err {e:.2e}")
    assert e < 1e-12
