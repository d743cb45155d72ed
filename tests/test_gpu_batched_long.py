"""Batched systems of more than 8192 rows, with helpers and without: the same bits."""
import re

import numpy as np
import pytest
import torch

import paper_2405_05865_amd as msp

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def _psd(n):
    p = torch.from_numpy(np.random.default_rng(n).standard_normal((n, 5))).to(DEV)
    a = torch.exp(-0.5 * torch.cdist(p, p) ** 2).float()
    return ((a + a.T) / 2).contiguous()


# last chunks of one row and whole chunks; beside a short system
@pytest.mark.parametrize("n,k", [(8193, 3), (9217, 1), (9216, 16)])
def test_long_systems(n, k, monkeypatch, capfd):
    print(f"case batched long n={n} k={k}", flush=True)
    monkeypatch.setenv("MSP_LOG", "1")
    s, lam, tol = 40, 0.5, 1e-9
    args = []
    for m in (n, 300):
        A = _psd(m)
        rows, signs, Y = msp.sketch(A, s, 8, 5)
        P = msp.Precond("psd", rows, signs, Y, lam, None, 4 * s, 8, 6, A=A)
        args.append((P, A, None, torch.from_numpy(np.random.default_rng([m, k]).standard_normal((k, m))).to(DEV)))
    out = {}
    for teams in (1, 0):
        capfd.readouterr()
        Xs, infos = msp.solve_batched(args, tol=tol, refine=1, batch_teams=teams, profile=1)
        helped = [int(v) for v in re.findall(r"slices helped (\d+)", capfd.readouterr().err)]
        assert len(helped) == 2 and (max(helped) > 0) == bool(teams), helped
        assert all(i["status"] == "MSP_OK" for i in infos), infos
        out[teams] = Xs
    for (P, A, _, B), X, Y in zip(args, out[1], out[0]):
        assert torch.equal(X, Y)
        a = A.double()
        for j in range(k):
            # the solver's own criterion, recomputed
            assert (a @ X[j] + lam * X[j] - B[j]).norm() <= 1.01 * tol * B[j].norm()
