"""Inner solves whose blocks do not meet: one block solves alone, with the same bits."""
import re

import numpy as np
import pytest
import torch

import paper_2405_05865_amd as msp
from oracle import msp as omsp

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")

# every number of 64-column chunks with every number of rows per wavefront and columns per
# group, full and partial last groups, and several launches per solve
SHAPES = [(200, 1), (256, 8), (250, 11), (256, 32), (256, 33), (512, 2), (500, 3), (512, 7), (512, 13), (512, 24),
          (375, 64), (1024, 1), (700, 2)]


def _bits(P, A, B, opts, monkeypatch, capfd):
    runs = []
    for wait in (None, "-1", "0"):  # the built-in time, no wait at all, and one that may run out anywhere
        if wait is None:
            monkeypatch.delenv("MSP_INNER_WAIT_MS", raising=False)
        else:
            monkeypatch.setenv("MSP_INNER_WAIT_MS", wait)
        capfd.readouterr()
        X, info = msp.solve(P, A, B, **opts)
        assert info["status"] == "MSP_OK", info
        alone = sum(int(v) for v in re.findall(r"\] (\d+) inner solves of column groups by one block", capfd.readouterr().err))
        runs.append((X, info, alone))
    assert runs[1][2] > 0
    for X, info, _ in runs[1:]:
        assert torch.equal(X, runs[0][0])
        for f in ("outer_iters", "inner_iters", "level3_iters", "rel_residual_max"):
            assert info[f] == runs[0][1][f], f


@pytest.mark.parametrize("s,k", SHAPES)
def test_one_block_alone_gives_the_same_bits(s, k, monkeypatch, capfd):
    print(f"case one block alone s={s} k={k}", flush=True)
    monkeypatch.setenv("MSP_LOG", "1")
    n, lam = s + 37, 0.5
    g = np.random.default_rng([s, k])
    p = g.standard_normal((n, 6))
    a = np.exp(-0.5 * ((p[:, None, :] - p[None, :, :]) ** 2).sum(2))
    A, B = torch.from_numpy((a + a.T) / 2).to(DEV), torch.from_numpy(g.standard_normal((k, n))).to(DEV)
    rows, signs, Y = msp.sketch(A, s, 8, 5)
    P = msp.Precond("psd", rows, signs, Y, lam, omsp.paper_lambda0(np.linalg.eigvalsh(a)[::-1], s // 2), n, 8, 6)
    _bits(P, A, B, dict(tol=1e-6), monkeypatch, capfd)
    A = torch.from_numpy(g.standard_normal((n, n)) / np.sqrt(n)).to(DEV)
    rows, signs, Y = msp.sketch(A, s, 8, 5)
    P = msp.Precond("general", rows, signs, Y, lam, float(torch.linalg.norm(A) ** 2 / s), n, 8, 6)
    _bits(P, A, B, dict(tol=1e-6, normal=1), monkeypatch, capfd)
