"""The inner solves that do not run as one launch, at sizes that reach them: one kernel per step
(PSD, up to 16 columns), two kernels per step (general, up to 16 columns), the generic step
(wider blocks), and each of them replayed as graphs; and one-launch solves of several launches
and of two columns per group. Against dense solutions and the generic iteration."""
import re

import numpy as np
import pytest
import torch

import paper_2405_05865_amd as msp

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")
LAM = 0.5


def _case(structure, s, k):
    n = s + 37
    g = np.random.default_rng([n, k])
    if structure == "psd":
        p = torch.from_numpy(g.standard_normal((n, 6))).to(DEV)
        A = torch.exp(-0.5 * torch.cdist(p, p) ** 2)
        A = ((A + A.T) / 2).contiguous()
        M = A
    else:
        A = torch.from_numpy(g.standard_normal((n, n)) / np.sqrt(n)).to(DEV)
        M = A.T.contiguous() @ A
    B = torch.from_numpy(g.standard_normal((k, n))).to(DEV)
    rows, signs, Y = msp.sketch(A, s, 8, 5)
    if structure == "psd":
        P = msp.Precond("psd", rows, signs, Y, LAM, None, n, 8, 6, A=A)
    else:
        P = msp.Precond("general", rows, signs, Y, LAM, float(n / s), n, 8, 6)
    want = torch.linalg.solve(M + LAM * torch.eye(n, dtype=torch.float64, device=DEV), B.T.contiguous()).T
    opts = dict(tol=1e-9) if structure == "psd" else dict(tol=1e-6, normal=1)
    return P, A, B, want, opts


def _check(X, info, want, B, tol):
    assert info["status"] == "MSP_OK", info
    # |x - x*| <= |r| / lam with |r| <= tol |b|; as much again for the dense solve's rounding
    assert torch.all((X - want).norm(dim=1) <= 2 * tol * B.norm(dim=1) / LAM)


# one kernel per step, then the generic step; one-launch solves with two columns per group of 4 and
# 8 chunks and of two and four launches
PSD = [(1100, 1), (1025, 2), (1100, 5), (1100, 16), (700, 3), (700, 16), (1100, 17), (700, 40),
       (256, 12), (512, 8), (512, 24), (375, 64)]


@pytest.mark.parametrize("s,k", PSD)
def test_psd_inner_solves(s, k):
    print(f"case routes psd s={s} k={k}", flush=True)
    P, A, B, want, opts = _case("psd", s, k)
    X, info = msp.solve(P, A, B, **opts)
    _check(X, info, want, B, opts["tol"])
    X0, info0 = msp.solve(P, A, B, level2_form=0, **opts)
    assert abs(info["outer_iters"] - info0["outer_iters"]) <= 2
    assert abs(info["inner_iters"] - info0["inner_iters"]) <= 0.05 * info0["inner_iters"] + 4
    X2, info2 = msp.solve(P, A, B, **opts)
    assert torch.equal(X, X2) and info2["inner_iters"] == info["inner_iters"]


# two kernels per step, the generic step, one-launch solves of two columns per group
GENERAL = [(700, 8), (600, 9), (600, 16), (1100, 1), (1100, 3), (700, 20), (256, 12), (512, 8)]


@pytest.mark.parametrize("s,k", GENERAL)
def test_level3_solves(s, k):
    print(f"case routes general s={s} k={k}", flush=True)
    P, A, B, want, opts = _case("general", s, k)
    X, info = msp.solve(P, A, B, **opts)
    _check(X, info, want, B, opts["tol"])
    X0, info0 = msp.solve(P, A, B, level3_kernels=0, **opts)
    assert abs(info["outer_iters"] - info0["outer_iters"]) <= 2
    assert abs(info["level3_iters"] - info0["level3_iters"]) <= 0.05 * info0["level3_iters"] + 8
    X2, info2 = msp.solve(P, A, B, **opts)
    assert torch.equal(X, X2) and info2["level3_iters"] == info["level3_iters"]


# the three kinds of step graphs
@pytest.mark.parametrize("structure,s,k,l3", [("psd", 700, 3, 2), ("psd", 1100, 1, 2), ("psd", 700, 40, 2),
                                              ("general", 700, 8, 2), ("general", 1100, 1, 2),
                                              ("general", 700, 20, 2), ("general", 64, 1, 0)])
def test_replayed_steps_give_the_same_bits(structure, s, k, l3, monkeypatch, capfd):
    print(f"case replayed steps {structure} s={s} k={k} level3_kernels={l3}", flush=True)
    monkeypatch.setenv("MSP_LOG", "1")
    P, A, B, want, opts = _case(structure, s, k)
    runs = []
    for graph in (0, 1, 1, 0):
        capfd.readouterr()
        X, info = msp.solve(P, A, B, use_graph=graph, level3_kernels=l3, **opts)
        _check(X, info, want, B, opts["tol"])
        replays = sum(int(v) for v in re.findall(r"(\d+) replays", capfd.readouterr().err))
        assert (replays > 1) == bool(graph)
        runs.append((X, info))
    for X, info in runs[1:]:
        assert torch.equal(X, runs[0][0])
        for f in ("outer_iters", "inner_iters", "level3_iters"):
            assert info[f] == runs[0][1][f]
