"""No result depends on what a workspace or an output buffer held before: every entry point twice,
with every new device buffer full of zeros and full of NaN (all bits set), to the same bits."""
import numpy as np
import pytest
import torch

import paper_2405_05865_amd as msp

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def _rng(*seed):
    return np.random.default_rng(list(seed))


def _psd(n):
    p = torch.from_numpy(_rng(n).standard_normal((n, 6))).to(DEV)
    a = torch.exp(-0.5 * torch.cdist(p, p) ** 2)
    return (a + a.T) / 2


def _gen(m, n):
    g = _rng(m, n)
    u = torch.linalg.qr(torch.from_numpy(g.standard_normal((m, n))))[0]
    v = torch.linalg.qr(torch.from_numpy(g.standard_normal((n, n))))[0]
    return ((u * torch.linspace(1, 4, n, dtype=torch.float64)) @ v).to(DEV).contiguous()


def _rhs(k, n):
    return torch.from_numpy(_rng(k, n, 1).standard_normal((k, n))).to(DEV)


def _handle(A, s, lam, structure):
    rows, signs, Y = msp.sketch(A, s, min(8, s), 5)
    n = A.shape[1]
    if structure == "psd":
        return msp.Precond("psd", rows, signs, Y, lam, -1.0, min(n, 4 * s), min(8, s), 6, A=A)
    return msp.Precond("general", rows, signs, Y, lam, 8.0 * n / s, min(n, 4 * s), min(8, s), 6)


def _solve(structure, n, s, k, lo=None, **opts):
    normal = opts.get("normal", 1)
    A = _psd(n) if structure == "psd" else _gen(n, n)
    if lo == torch.float32:
        A = A.float()
    lam = 0.5 if structure == "psd" or normal else 0.0
    P = _handle(A, s, lam, structure)
    X, info = msp.solve(P, A, _rhs(k, n), A_lo=None if lo is None else A.to(lo), tol=1e-6, inner_tol=1e-8,
                        level3_tol=1e-8, refine=0 if lo is None else 1, **opts)
    assert info["status"] == "MSP_OK", info
    return [X, info["outer_iters"], info["inner_iters"], info["level3_iters"], info["rel_residual_max"]]


def _setup(dtype, n, s):
    A = _psd(n).to(dtype)
    rows, signs, Y = msp.sketch(A, s, 8, 5)
    P = msp.Precond("psd", rows, signs, Y, 0.5, -1.0, min(n, 4 * s), 8, 6, A=A)
    G = msp.Precond("general", rows, signs, Y, 0.5, 1.0, min(n, 4 * s), 8, 6)
    return [rows, signs, Y, P.lam0, *P.factors()[:2], *G.factors()[1:]]


def _batched(s, dtype):
    systems, grads = [], []
    for n in (300, 555):
        A = _psd(n).to(dtype)
        systems.append((_handle(A, s, 0.5, "psd"), A, None, _rhs(5, n)))
        grads.append(_rhs(5, n) + 1.0)
    opts = dict(tol=1e-8, refine=int(dtype == torch.float32))
    Xs, infos = msp.solve_batched(systems, **opts)
    dBs, dl, dAs, _ = msp.solve_batched_backward(systems, Xs, grads, want_dA=True, **opts)
    return [*Xs, *dBs, *dl, *dAs, *[i["outer_iters"] for i in infos]]


def _backward(k):
    A = _psd(300)
    P = _handle(A, 40, 0.5, "psd")
    X, _ = msp.solve(P, A, _rhs(k, 300), tol=1e-8)
    return [X, *msp.solve_backward(P, A, X, _rhs(k, 300) + 1.0, want_dA=True, tol=1e-8)[:3]]


def _trace(kind):
    probes = msp.gaussian_probes(200, 9, 3)
    if kind == "effdim":
        A = _psd(200)
        return list(msp.effective_dimension(_handle(A, 24, 0.5, "psd"), A, probes, 0.5, tol=1e-6)[:2])
    A = _gen(200, 200)
    P = _handle(A, 24, 0.5, "general")
    opts = dict(tol=1e-6, normal=1)
    if kind == "orlicz":
        return list(msp.orlicz(P, A, probes, [1.0], [1.0], h=3.0, **opts)[:2])
    return list(msp.schatten(P, A, probes, p=1.0, h=3.0, **opts)[:2])


def _lstsq(k, dtype):
    n, d = 900, 60
    A = _gen(n, d).to(dtype)
    rows, signs, At = msp.left_sketch(A, 240, 8, 7)
    s_rows, s_signs, Y = msp.sketch(At, 24, 8, 5)
    P = msp.Precond("general", s_rows, s_signs, Y, 0.0, 20.0, 60, 8, 6)
    X, info = msp.lstsq(P, At, A, _rhs(k, n), tol=1e-8, inner_tol=1e-8, level3_tol=1e-8)
    assert info["status"] == "MSP_OK", info
    return [rows, signs, At, X, info["outer_iters"]]


CASES = {
    **{f"setup {d} n={n} s={s}": (_setup, d, n, s) for d in (torch.float64, torch.float32) for n, s in ((300, 40), (513, 130))},
    **{f"psd n={n} s={s} k={k} form={f}": (_solve, "psd", n, s, k, None, f)
       for n, s, k in ((300, 5, 2), (300, 40, 1), (400, 130, 9), (400, 200, 20), (1200, 1030, 3), (1300, 300, 2))
       for f in (0, 1, 2)},
    **{f"psd refine {lo} k={k}": (_solve, "psd", 300, 40, k, lo, 1) for lo in (torch.float32, torch.bfloat16) for k in (1, 3, 12)},
    **{f"general n={n} s={s} k={k} form={f} normal={nm}": (_solve, "general", n, s, k, None, f, nm)
       for n, s, k in ((300, 5, 2), (300, 40, 1), (400, 130, 9), (400, 200, 20), (700, 512, 8), (2100, 40, 3))
       for f in (0, 1, 2) for nm in (0, 1) if f or (nm and n < 2000)},
    **{f"general refine k={k} normal={nm}": (_solve, "general", 300, 40, k, torch.float32, 1, nm) for k in (1, 12) for nm in (0, 1)},
    "general generic level-3 step": (_solve, "general", 400, 130, 9, None, 1, 1, 0),
    "autotuned sweep": (_solve, "psd", 600, 40, 12, None, 1, 1, 2, 1),
    **{f"batched s={s} {d}": (_batched, s, d) for s in (40, 270) for d in (torch.float64, torch.float32)},
    **{f"backward k={k}": (_backward, k) for k in (1, 9)},
    **{f"trace {k}": (_trace, k) for k in ("schatten", "orlicz", "effdim")},
    "kyfan": (lambda: [v for r in msp.kyfan(_gen(300, 200), 5) for v in (r if isinstance(r, list) else [r])],),
    **{f"lstsq k={k} {d}": (_lstsq, k, d) for k in (1, 9) for d in (torch.float64, torch.float32)},
}


def _call(f, *args):
    if f is _solve:
        structure, n, s, k, lo, form, *rest = args
        opts = dict(level2_form=form)
        if structure == "general":
            opts["normal"] = rest[0] if rest else 1
            if len(rest) > 1:
                opts["level3_kernels"] = rest[1]
        if len(rest) > 2:
            opts["autotune"] = rest[2]
        return _solve(structure, n, s, k, lo, **opts)
    return f(*args)


@pytest.mark.parametrize("name", list(CASES))
def test_results_do_not_depend_on_old_memory(name, monkeypatch):
    print("case old memory", name, flush=True)
    real, fill = torch.empty, [0]

    def empty(*a, **kw):
        t = real(*a, **kw)
        if t.is_cuda:
            t.view(torch.uint8).fill_(fill[0]) if t.dim() else t.fill_(0)
        return t

    runs = []
    for v in (0, 255):
        fill[0] = v
        monkeypatch.setattr(torch, "empty", empty)
        try:
            runs.append(_call(*CASES[name]))
        finally:
            monkeypatch.setattr(torch, "empty", real)
    for a, b in zip(*runs):
        assert torch.equal(a, b) if isinstance(a, torch.Tensor) else (a == b), name
