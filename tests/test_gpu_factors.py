"""Factors of the preconditioner at sizes around the tiles of their kernels, against numpy."""
import numpy as np
import pytest
import torch

import paper_2405_05865_amd as msp
from oracle import rng, sketch as osk

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


# pivot blocks of 32 (whole and short last ones), tiles of 64, row splits of the Gram product
@pytest.mark.parametrize("n,s,dtype", [(70, 9, torch.float64), (300, 31, torch.float64), (300, 32, torch.float64),
                                       (300, 33, torch.float32), (700, 64, torch.float64), (701, 65, torch.float64),
                                       (1500, 130, torch.float32), (5000, 200, torch.float64)])
def test_factors_at_tile_edges(n, s, dtype):
    print(f"case factors n={n} s={s} {dtype}", flush=True)
    g = np.random.default_rng([n, s])
    p = g.standard_normal((n, 5))
    a = np.exp(-0.5 * ((p[:, None, :] - p[None, :, :]) ** 2).sum(2)) if n <= 1500 else None
    if a is None:
        f = g.standard_normal((n, 40)) / np.sqrt(40)
        a = f @ f.T + 0.5 * np.eye(n)
    A = torch.from_numpy((a + a.T) / 2).to(DEV).to(dtype)
    rows, signs, Y = msp.sketch(A, s, 8, 3)
    lam, phi = 0.1, min(4 * s, n)
    P = msp.Precond("psd", rows, signs, Y, lam, None, phi, 8, 4, A=A)
    W, Minv, _ = P.factors()
    # the same factors from the device's own sketch in float64: only the factors' rounding differs
    y = Y.double().cpu().numpy()
    r, sg = rows.cpu().numpy(), signs.cpu().numpy()
    S = osk.dense_embedding(r, sg, s)
    w = S @ y
    w = (w + w.T) / 2
    # sums of up to n terms: |error| <= n eps sum |terms|
    eps = np.finfo(np.float64).eps
    assert np.all(np.abs(W.cpu().numpy() - w) <= n * eps * (np.abs(S) @ np.abs(y)).max())
    mu = 1e-9 * np.trace(w) / s
    ctc = y.T @ y
    deficit = float(A.double().diagonal().sum()) - float((np.linalg.inv(w + mu * np.eye(s)) * ctc).sum())
    want0 = 2.0 / (0.5 * s) * deficit
    kappa_w = np.linalg.cond(w + mu * np.eye(s))
    assert abs(P.lam0 - want0) <= 2.0 / (0.5 * s) * kappa_w * 1e-12 * np.abs(ctc).max() * s
    ri, si = rng.sketch_indices(4, n, phi, 8)
    z = osk.left_sketch(ri, si, phi, y)
    m2 = z.T @ z + (lam + P.lam0) * w
    m2 = (m2 + m2.T) / 2 + 1e-12 * np.trace(m2) / s * np.eye(s)
    got = Minv.cpu().numpy()
    want = np.linalg.inv(m2)
    # a relative perturbation of s eps in M becomes kappa(M) s eps in its inverse (and numpy's own)
    assert np.linalg.norm(got - want) <= 4 * np.linalg.cond(m2) * s * eps * np.linalg.norm(want)
    assert np.array_equal(got, got.T)
