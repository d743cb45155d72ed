"""Solves on several streams at once, beside a batch that fills the chip: the same bits as alone."""
import threading

import numpy as np
import pytest
import torch

import paper_2405_05865_amd as msp

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def _psd(n, dtype=torch.float64):
    p = torch.from_numpy(np.random.default_rng(n).standard_normal((n, 6))).to(DEV)
    a = torch.exp(-0.5 * torch.cdist(p, p) ** 2)
    return ((a + a.T) / 2).to(dtype).contiguous()


def _handle(A, s, lam):
    rows, signs, Y = msp.sketch(A, s, 8, 5)
    return msp.Precond("psd", rows, signs, Y, lam, None, min(4 * s, A.shape[0]), 8, 6, A=A)


def _rhs(k, n):
    return torch.from_numpy(np.random.default_rng([k, n]).standard_normal((k, n))).to(DEV)


def _jobs():
    jobs = []
    for n, s, k in ((1200, 256, 1), (1500, 512, 8), (900, 200, 20)):
        A, B = _psd(n), _rhs(k, n)
        P = _handle(A, s, 0.05)
        jobs.append(lambda P=P, A=A, B=B: [msp.solve(P, A, B, tol=1e-9)[0]])
    g = torch.from_numpy(np.random.default_rng(4).standard_normal((700, 700)) / np.sqrt(700)).to(DEV)
    rows, signs, Y = msp.sketch(g, 300, 8, 5)
    G, C = msp.Precond("general", rows, signs, Y, 0.5, 2.3, 700, 8, 6), _rhs(2, 700)
    jobs.append(lambda: [msp.solve(G, g, C, tol=1e-8, normal=1)[0]])
    systems = []
    for n in (2500, 1800, 1100):
        A = _psd(n, torch.float32)
        systems.append((_handle(A, 64, 0.05), A, None, _rhs(4, n)))
    jobs.append(lambda: msp.solve_batched(systems, tol=1e-9, refine=1)[0])
    return jobs


def test_concurrent_solves_give_the_same_bits():
    print("case concurrent solves on five streams", flush=True)
    jobs = _jobs()
    want = [job() for job in jobs]
    torch.cuda.synchronize()
    bad = []

    def work(i):
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(8):
                got = jobs[i]()
                torch.cuda.current_stream().synchronize()
                if not all(torch.equal(a, b) for a, b in zip(got, want[i])):
                    bad.append(i)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(jobs))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad, bad
