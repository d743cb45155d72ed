"""Blocks of more than sixteen right-hand sides on PSD systems whose level-2 operator is
ill-conditioned: a few eigenvalues from 1e6 to 1e2 above a floor. The inner iteration needs
direct products there; one that carries H p by a recurrence drifts and the solve stalls."""
import numpy as np
import pytest
import torch

import paper_2405_05865_amd as msp

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


# one block per column, groups of several blocks, two and four launches per inner solve
@pytest.mark.parametrize("s,k", [(64, 20), (128, 17), (256, 20), (256, 64), (512, 24), (375, 64)])
def test_wide_blocks_on_ill_conditioned_systems(s, k):
    print(f"case ill-conditioned s={s} k={k}", flush=True)
    n, lam, floor, tol = 1000, 1e-3, 0.1, 1e-9
    g = np.random.default_rng([n, s])
    q = torch.linalg.qr(torch.from_numpy(g.standard_normal((n, n))))[0]
    e = torch.full((n,), floor, dtype=torch.float64)
    e[:s // 2] = torch.logspace(6, 2, s // 2, dtype=torch.float64)
    a = (q * e) @ q.T
    A = ((a + a.T) / 2).to(DEV).contiguous()
    b = g.standard_normal((k, n))
    B = torch.from_numpy(b).to(DEV)
    rows, signs, Y = msp.sketch(A, s, 8, 5)
    P = msp.Precond("psd", rows, signs, Y, lam, None, min(4 * s, n), 8, 6, A=A)
    X, info = msp.solve(P, A, B, tol=tol, max_outer=300)
    assert info["status"] == "MSP_OK", info
    # the operator through the sketch: the same iteration with direct products
    X0, info0 = msp.solve(P, A, B, tol=tol, max_outer=300, level2_form=0)
    assert info["outer_iters"] <= 2 * info0["outer_iters"], (info, info0)
    want = np.linalg.solve(A.cpu().numpy() + lam * np.eye(n), b.T).T
    x = X.cpu().numpy()
    for j in range(k):
        # |x - x*| <= |r| / (floor + lam) with |r| <= tol |b|; as much again for the dense solve
        assert np.linalg.norm(x[j] - want[j]) <= 2 * tol * np.linalg.norm(b[j]) / (floor + lam)
