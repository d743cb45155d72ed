"""Sweeps over matrices whose rows are not 16-byte aligned, against dense solutions."""
import numpy as np
import pytest
import torch

import paper_2405_05865_amd as msp
import workloads as W
from oracle import dense
from oracle import msp as omsp

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def _offset_view(a, dtype, offset, pad):
    """a as a view `offset` elements into a buffer with `pad` extra columns; the rest is NaN."""
    m, n = a.shape
    ld = n + pad
    buf = torch.full((offset + m * ld,), float("nan"), dtype=dtype, device=DEV)
    v = buf[offset:].as_strided((m, n), (ld, 1), offset)
    v.copy_(torch.from_numpy(a).to(DEV).to(dtype))
    return v


# one, two and four columns take the vector sweep, 8, 16 and 33 the matrix cores; the odd
# leading dimensions and bases break the 16-byte alignment in every storage type
@pytest.mark.parametrize("k", [1, 2, 4, 8, 16, 33])
@pytest.mark.parametrize("dtype,offset,pad", [(torch.float64, 1, 0), (torch.float64, 0, 2), (torch.float32, 3, 1)])
def test_psd_solve_at_any_alignment(k, dtype, offset, pad):
    print(f"case alignment k={k} {dtype} offset={offset} pad={pad}", flush=True)
    n, s, lam, tol = 515, 64, 0.5, 1e-10
    a, eigs, _ = W.psd_outlier(n, 16, config_id=7)
    lam0 = omsp.paper_lambda0(eigs, s // 2)
    A = _offset_view(a, dtype, offset, pad)
    a_lo = A.double().cpu().numpy()
    a_lo = (a_lo + a_lo.T) / 2
    b = np.random.default_rng(k).standard_normal((k, n))
    rows, signs, Y = msp.sketch(A, s, 8, 51)
    P = msp.Precond("psd", rows, signs, Y, lam, lam0, 4 * s, 8, 52)
    X, info = msp.solve(P, A, torch.from_numpy(b).to(DEV), tol=tol, refine=0 if dtype == torch.float64 else 1)
    assert info["status"] == "MSP_OK", info
    x = X.cpu().numpy()
    for j in range(k):
        # |x - x*| <= |r| / (lam_min + lam) <= tol |b| / lam, and |x*| >= |b| / (lam_max + lam)
        xs = dense.solve_psd(a_lo, b[j], lam)
        assert np.linalg.norm(x[j] - xs) <= 2 * tol * np.linalg.norm(b[j]) / lam


@pytest.mark.parametrize("k", [1, 4, 12])
def test_bf16_sweeps_at_any_alignment(k):
    # bf16 sweeps pay off where lam dominates the rounding of A: a kernel matrix and lam = 0.5
    print(f"case bf16 alignment k={k}", flush=True)
    n, s, lam, tol = 515, 64, 0.5, 1e-10
    p = np.random.default_rng(5).standard_normal((n, 8))
    a = np.exp(-0.5 * ((p[:, None, :] - p[None, :, :]) ** 2).sum(2))
    A_lo = _offset_view(a, torch.bfloat16, 5, 2)
    A = _offset_view(a, torch.float64, 5, 2)
    b = np.random.default_rng(k).standard_normal((k, n))
    rows, signs, Y = msp.sketch(A_lo, s, 8, 51)
    P = msp.Precond("psd", rows, signs, Y, lam, omsp.paper_lambda0(np.linalg.eigvalsh(a)[::-1], s // 2), 4 * s, 8, 52)
    X, info = msp.solve(P, A, torch.from_numpy(b).to(DEV), A_lo=A_lo, tol=tol, refine=1)
    assert info["status"] == "MSP_OK", info
    for j in range(k):
        xs = dense.solve_psd(a, b[j], lam)
        assert np.linalg.norm(X[j].cpu().numpy() - xs) <= 2 * tol * np.linalg.norm(b[j]) / lam


@pytest.mark.parametrize("k", [1, 8, 20])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_ridge_at_any_alignment(k, dtype):
    print(f"case ridge alignment k={k} {dtype}", flush=True)
    m, n, s, lam, tol = 413, 301, 32, 1.0, 1e-10
    g = np.random.default_rng(3)
    a = g.standard_normal((m, n)) / np.sqrt(n)
    A = _offset_view(a, dtype, 1, 0)
    a64 = A.double().cpu().numpy()
    sv = np.linalg.svd(a64, compute_uv=False)
    c = g.standard_normal((k, n))
    rows, signs, Y = msp.sketch(A, s, 8, 61)
    P = msp.Precond("general", rows, signs, Y, lam, omsp.paper_lambda0(sv ** 2, s // 2), 4 * s, 8, 62)
    X, info = msp.solve(P, A, torch.from_numpy(c).to(DEV), normal=1, tol=tol, refine=1)
    assert info["status"] == "MSP_OK", info
    xs = np.linalg.solve(a64.T @ a64 + lam * np.eye(n), c.T).T
    # the smallest eigenvalue of the operator is at least lam = 1
    for j in range(k):
        assert np.linalg.norm(X[j].cpu().numpy() - xs[j]) <= 2 * tol * np.linalg.norm(c[j])
