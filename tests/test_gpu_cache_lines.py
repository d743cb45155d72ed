"""Level-1 sweeps on both sides of the sizes at which their loads leave the caches and their
tiles grow, against products formed by the test itself."""
import pytest
import torch

import paper_2405_05865_amd as msp

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


# lower triangle (k = 1): 249, 251 and 301 MB; whole matrix (k = 3): 279 and 281 MB
@pytest.mark.parametrize("n,k,dtype", [(8080, 1, torch.float64), (8110, 1, torch.float64), (8886, 1, torch.float64),
                                       (11468, 1, torch.float32), (12564, 1, torch.float32),
                                       (6047, 3, torch.float64), (6073, 3, torch.float64)])
def test_solve_around_the_cache_size(n, k, dtype):
    print(f"case cache size n={n} k={k} {dtype}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(n)
    s, lam, tol = 64, 0.5, 1e-10
    U = torch.randn(n, 16, generator=g, device=DEV, dtype=torch.float64)
    A = U @ U.T * (40.0 / n)
    A.diagonal().add_(1.0)
    A = ((A + A.T) / 2).to(dtype)
    B = torch.randn(k, n, generator=g, device=DEV, dtype=torch.float64)
    rows, signs, Y = msp.sketch(A, s, 8, 51)
    P = msp.Precond("psd", rows, signs, Y, lam, float(s), 4 * s, 8, 52)
    X, info = msp.solve(P, A, B, tol=tol, refine=0 if dtype == torch.float64 else 1)
    assert info["status"] == "MSP_OK", info
    A64 = A.double()
    for j in range(k):
        r = B[j] - (A64 @ X[j] + lam * X[j])
        assert float(r.norm() / B[j].norm()) <= 1.01 * tol
