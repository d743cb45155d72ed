"""The batched solve at the edges of its tiles: sketch sizes around the 16-element blocks, the
32-row tiles and the 256-element limit of the level-2 solve on LDS (and the general path behind
it), systems around the 256-row chunks, odd rows and pitches, one to sixteen columns, each
against a dense solve and, with helpers off, the same bits."""
import numpy as np
import pytest
import torch

import paper_2405_05865_amd as msp
import workloads as W
from oracle import dense
from oracle import msp as omsp

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def _system(n, s, cid, dtype, pad):
    pts = W.rbf_points(n, 4, cid)
    a = W.rbf_matrix(pts, lengthscale=0.8, dtype=dtype)
    a64 = a.astype(np.float64)
    lam0 = omsp.paper_lambda0(np.linalg.eigvalsh(a64)[::-1], max(1, s // 2))
    buf = torch.zeros((n, n + pad), dtype=torch.float32 if dtype == np.float32 else torch.float64, device=DEV)
    buf[:, :n] = torch.from_numpy(a).to(DEV)
    A = buf[:, :n]
    rows, signs, Y = msp.sketch(A, s, min(8, s), 71 + cid, y_dtype=A.dtype)
    P = msp.Precond("psd", rows, signs, Y, 1e-2, lam0, min(4 * s, n), min(8, s), 81 + cid)
    return a64, P, A


@pytest.mark.parametrize("sizes,k,dtype", [
    ([(255, 2), (256, 15), (257, 16), (258, 17), (511, 31)], 16, np.float64),
    ([(513, 33), (300, 63), (301, 64), (302, 65)], 1, np.float32),
    ([(600, 143), (601, 191), (602, 193)], 5, np.float32),
    ([(700, 254), (701, 255), (769, 256), (703, 257)], 15, np.float64),
    ([(768, 255), (1025, 256), (770, 258)], 16, np.float32),
])
def test_batched_edges(sizes, k, dtype):
    lam, args, mats, Bs = 1e-2, [], [], []
    for i, (n, s) in enumerate(sizes):
        print("case batched edges", n, s, k, dtype.__name__, flush=True)
        a64, P, A = _system(n, s, 40 + i, dtype, pad=i % 3)
        Bm = W.gaussian((k, n), 900 + i)
        mats.append(a64)
        Bs.append(Bm)
        args.append((P, A, None, torch.from_numpy(Bm).to(DEV)))
    opts = dict(tol=1e-10, refine=1 if dtype == np.float32 else 0, max_outer=5000)
    Xs, infos = msp.solve_batched(args, **opts)
    X0, infos0 = msp.solve_batched(args, batch_teams=0, **opts)
    for a64, Bm, X, Y, info, info0 in zip(mats, Bs, Xs, X0, infos, infos0):
        assert info["status"] == "MSP_OK" and info0["status"] == "MSP_OK", (info, info0)
        x = X.cpu().numpy()
        assert np.array_equal(x, Y.cpu().numpy())
        for j in range(k):
            # the solver's own criterion, recomputed in FP64
            assert dense.rel_residual_psd(a64, x[j], Bm[j], lam) <= 1.01e-10
