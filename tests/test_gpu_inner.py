"""Inner solves that run as one launch: sizes around the kernel's tiles and column groups,
against dense solutions, and the per-step kernels as the way out when its blocks cannot meet."""
import numpy as np
import pytest
import torch

import paper_2405_05865_amd as msp
from oracle import msp as omsp

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")
TOL = 1e-10


def _psd(n, s, k, lam=0.5):
    g = np.random.default_rng([n, s, k])
    p = g.standard_normal((n, 6))
    a = np.exp(-0.5 * ((p[:, None, :] - p[None, :, :]) ** 2).sum(2))
    a = (a + a.T) / 2
    b = g.standard_normal((k, n))
    A, B = torch.from_numpy(a).to(DEV), torch.from_numpy(b).to(DEV)
    rows, signs, Y = msp.sketch(A, s, min(8, s), 5)
    lam0 = omsp.paper_lambda0(np.linalg.eigvalsh(a)[::-1], max(1, s // 2))
    P = msp.Precond("psd", rows, signs, Y, lam, lam0, min(4 * s, n), 8, 6)
    want = np.linalg.solve(a + lam * np.eye(n), b.T).T
    return P, A, B, b, want, lam


def _ridge(n, s, k, lam=0.5):
    g = np.random.default_rng([n, s, k])
    a = g.standard_normal((n, n)) / np.sqrt(n)
    b = g.standard_normal((k, n))
    A, B = torch.from_numpy(a).to(DEV), torch.from_numpy(b).to(DEV)
    rows, signs, Y = msp.sketch(A, s, min(8, s), 5)
    lam0 = omsp.paper_lambda0(np.linalg.svd(a, compute_uv=False) ** 2, max(1, s // 2))
    P = msp.Precond("general", rows, signs, Y, lam, lam0, min(4 * s, n), 8, 6)
    want = np.linalg.solve(a.T @ a + lam * np.eye(n), b.T).T
    return P, A, B, b, want, lam


def _check(X, want, b, lam):
    # |x - x*| <= |r| / lam with |r| <= TOL |b|; as much again for the dense solve's rounding
    x = X.cpu().numpy()
    for j in range(len(b)):
        assert np.linalg.norm(x[j] - want[j]) <= 2 * TOL * np.linalg.norm(b[j]) / lam


# one block (s <= 128), rows per block and chunk counts (129, 256, 257, 512, 513, 1024), column
# groups of one, two and four with full and partial last groups, and launches one after another
SIZES = [(8, 1), (63, 2), (64, 17), (65, 1), (128, 3), (129, 1), (200, 9), (256, 8), (256, 33), (257, 4), (320, 5),
         (512, 1), (500, 13), (513, 2), (700, 3), (1024, 1)]


@pytest.mark.parametrize("s,k", SIZES)
def test_psd_inner_solve_in_one_launch(s, k):
    print(f"case one-launch level 2 s={s} k={k}", flush=True)
    P, A, B, b, want, lam = _psd(max(200, s + 37), s, k)
    X, info = msp.solve(P, A, B, tol=TOL)
    assert info["status"] == "MSP_OK", info
    _check(X, want, b, lam)
    # the operator through the sketch takes the generic steps: the same iteration
    X0, info0 = msp.solve(P, A, B, tol=TOL, level2_form=0)
    assert abs(info["outer_iters"] - info0["outer_iters"]) <= 2
    assert abs(info["inner_iters"] - info0["inner_iters"]) <= 0.05 * info0["inner_iters"] + 4
    X2, info2 = msp.solve(P, A, B, tol=TOL)
    assert torch.equal(X, X2) and info2["inner_iters"] == info["inner_iters"]


@pytest.mark.parametrize("s,k", SIZES)
def test_level3_solves_in_one_launch(s, k):
    print(f"case one-launch level 3 s={s} k={k}", flush=True)
    P, A, B, b, want, lam = _ridge(max(200, s + 37), s, k)
    X, info = msp.solve(P, A, B, tol=TOL, normal=1)
    assert info["status"] == "MSP_OK", info
    _check(X, want, b, lam)
    X0, info0 = msp.solve(P, A, B, tol=TOL, normal=1, level3_kernels=0)
    assert abs(info["outer_iters"] - info0["outer_iters"]) <= 2
    assert abs(info["level3_iters"] - info0["level3_iters"]) <= 0.05 * info0["level3_iters"] + 8
    X2, info2 = msp.solve(P, A, B, tol=TOL, normal=1)
    assert torch.equal(X, X2) and info2["level3_iters"] == info["level3_iters"]


@pytest.mark.parametrize("k", [1, 20])
def test_inner_solve_that_gives_up_takes_the_steps(k, monkeypatch):
    print(f"case one-launch gives up k={k}", flush=True)
    s, n = 200, 300
    P, A, B, b, want, lam = _psd(n, s, k)
    Pg, Ag, Bg, bg, wantg, lamg = _ridge(n, s, k)
    monkeypatch.setenv("MSP_INNER_WAIT_MS", "-1")
    X, info = msp.solve(P, A, B, tol=TOL)
    assert info["status"] == "MSP_OK", info
    _check(X, want, b, lam)
    X, info = msp.solve(Pg, Ag, Bg, tol=TOL, normal=1)
    assert info["status"] == "MSP_OK", info
    _check(X, wantg, bg, lamg)
    monkeypatch.delenv("MSP_INNER_WAIT_MS")
    X, info = msp.solve(P, A, B, tol=TOL)
    assert info["status"] == "MSP_OK", info
    _check(X, want, b, lam)


def test_zero_columns_and_iteration_caps_in_one_launch():
    print("case one-launch zero column and caps", flush=True)
    P, A, B, b, want, lam = _psd(300, 150, 5)
    B[2] = 0.0
    X, info = msp.solve(P, A, B, tol=TOL)
    assert info["status"] == "MSP_OK" and torch.all(X[2] == 0.0)
    want[2], b[2] = 0.0, 0.0
    _check(X, want, b, lam)
    X, info = msp.solve(P, A, B, tol=TOL, max_inner=1)  # every inner solve stops at its cap
    assert info["inner_iters"] <= info["outer_iters"] + info["restarts"] + 1
    _check(X, want, b, lam)


# level-1 vectors at the limits of the one-block steps: 2048 elements, 8192 over the columns
@pytest.mark.parametrize("n,k", [(2048, 4), (2048, 5), (2049, 1), (1024, 8), (910, 9), (65, 16), (64, 3)])
def test_steps_of_short_vectors(n, k):
    print(f"case short vectors n={n} k={k}", flush=True)
    s = max(8, min(64, n // 4))
    P, A, B, b, want, lam = _ridge(n, s, k)
    X, info = msp.solve(P, A, B, tol=TOL, normal=1)
    assert info["status"] == "MSP_OK", info
    _check(X, want, b, lam)
    P, A, B, b, want, lam = _psd(n, s, k)
    X, info = msp.solve(P, A, B, tol=TOL)
    assert info["status"] == "MSP_OK", info
    _check(X, want, b, lam)
