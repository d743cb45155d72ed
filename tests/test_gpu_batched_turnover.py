"""A batch of more systems than compute units: a unit whose system is finished goes to the next
system at once."""
import time

import numpy as np
import pytest
import torch

import paper_2405_05865_amd as msp

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def test_a_finished_system_makes_room():
    n, s, k, lam = 64, 8, 256, 0.5  # sixteen launches of sixteen columns
    nsys = torch.cuda.get_device_properties(0).multi_processor_count + 64
    print(f"case batch turnover {nsys} systems of {n}", flush=True)
    g = np.random.default_rng(3)
    p = g.standard_normal((n, 4))
    a = np.exp(-0.5 * ((p[:, None, :] - p[None, :, :]) ** 2).sum(2))
    A = torch.from_numpy((a + a.T) / 2).to(DEV)
    rows, signs, Y = msp.sketch(A, s, 8, 5)
    P = msp.Precond("psd", rows, signs, Y, lam, 1.0, n, 8, 6)
    args = [(P, A, None, torch.from_numpy(g.standard_normal((k, n))).to(DEV)) for _ in range(nsys)]

    def once(teams):
        torch.cuda.synchronize()
        t = time.perf_counter()
        Xs, infos = msp.solve_batched(args, tol=1e-8, batch_teams=teams)
        torch.cuda.synchronize()
        assert all(i["status"] == "MSP_OK" for i in infos)
        return time.perf_counter() - t, Xs

    best = {0: 1e9, 1: 1e9}
    for _ in range(4):
        for teams in (0, 1):
            t, Xs = once(teams)
            best[teams] = min(best[teams], t)
    print(f"without teams {1e3 * best[0]:.2f} ms, with teams {1e3 * best[1]:.2f} ms", flush=True)
    for i in (0, nsys - 1):
        want = np.linalg.solve(a + lam * np.eye(n), args[i][3].cpu().numpy().T).T
        # |x - x*| <= |r| / lam with |r| <= tol |b|; as much again for the dense solve's rounding
        assert np.linalg.norm(Xs[i].cpu().numpy() - want) <= 2e-8 * np.linalg.norm(want) * (1 + np.linalg.norm(a, 2) / lam)
    # a wait for the systems that have not started would cost a millisecond in every launch
    assert best[1] <= best[0] + 0.5e-3 * (k // 16)
