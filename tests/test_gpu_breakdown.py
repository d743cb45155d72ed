"""A column whose direction is not finite stops as a breakdown and keeps its iterate, whatever
kernel takes the step; the other columns of the block go on."""
import numpy as np
import pytest
import torch

import paper_2405_05865_amd as msp

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


# the one-block steps (short vectors: in registers, and in several passes) and the launches of
# longer ones
@pytest.mark.parametrize("n,k", [(96, 3), (2000, 4), (1500, 3), (2049, 3)])
def test_a_breakdown_keeps_the_iterate(n, k):
    print(f"case breakdown n={n} k={k}", flush=True)
    lam, s, tol = 0.5, 24, 1e-10
    g = np.random.default_rng([n, k])
    a = g.standard_normal((n, n)) / np.sqrt(n)
    c = g.standard_normal((k, n))
    c[1, 7] = np.nan  # no direction of this column is finite: its iterate is the initial zero
    A, C = torch.from_numpy(a).to(DEV), torch.from_numpy(c).to(DEV)
    rows, signs, Y = msp.sketch(A, s, 8, 5)
    lam0 = float(np.linalg.norm(a) ** 2 / s)
    P = msp.Precond("general", rows, signs, Y, lam, lam0, 4 * s, 8, 6)
    X, info = msp.solve(P, A, C, tol=tol, normal=1)
    x = X.cpu().numpy()
    assert np.array_equal(x[1], np.zeros(n))
    for j in range(k):
        if j != 1:
            # |x - x*| <= |r| / lam with |r| <= tol |c|; as much again for the dense solve's rounding
            want = np.linalg.solve(a.T @ a + lam * np.eye(n), c[j])
            assert np.linalg.norm(x[j] - want) <= 2 * tol * np.linalg.norm(c[j]) / lam
