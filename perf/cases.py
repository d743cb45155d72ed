"""The work that a user of this package has it do, as cases that can be timed and checked.

Each case is a dict of plain values. ``prepare`` makes what a program has in hand before the
call, ``run`` makes one pass through the public entry points, ``work`` states the bytes and
operations that the pass cannot do without, and ``exact`` gives the same results from plain
dense linear algebra in 64 bits.

Kinds
  path      one whole solve from the matrix: sketch, preconditioner, two-level iteration
  solve     the PSD iteration on a prepared handle (Gaussian-process / kernel systems)
  sketch    S and Y = A S^T
  precond   the Nystrom handle and its inner factors from a sketch
  ridge     (A^T A + lam I) X = C through the three-level iteration on a prepared handle
  lstsq     tall least squares: sketched A~, its handle, and the preconditioned iteration
  schatten  the quadrature nodes of a Schatten-norm estimate
  batched   many uneven PSD systems in one launch, and their adjoints
  backward  a differentiable solve: forward and the gradients of A, B and lam
"""
import math

import numpy as np
import torch

import paper_2405_05865_amd as msp

_DT = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16}
_SIZE = {"f64": 8, "f32": 4, "bf16": 2}
_GAMMA = 8
_DEV = "cuda:0"


def listed():
    return [
        # a single small system with a few large eigenvalues: the whole call, bound by latency
        {"name": "path_n1024", "kind": "path", "n": 1024, "s": 64, "k": 1, "outliers": 32},
        # the Gaussian-process system at full size, one right-hand side, a handle in hand
        {"name": "solve_f64_n32768", "kind": "solve", "n": 32768, "s": 512, "k": 1, "a": "f64"},
        # sixteen right-hand sides as one block, a size off every tile edge
        {"name": "solve_block16_n10007", "kind": "solve", "n": 10007, "s": 320, "k": 16, "a": "f64"},
        # the same system stored in 32 bits with FP64 refinement
        {"name": "solve_f32_n12000", "kind": "solve", "n": 12000, "s": 384, "k": 1, "a": "f32"},
        # the sparse sketch of the full-size matrix
        {"name": "sketch_f64_n32768", "kind": "sketch", "m": 32768, "n": 32768, "s": 512, "a": "f64"},
        # the PSD handle at full size, lam0 estimated on the device
        {"name": "precond_psd_n32768", "kind": "precond", "psd": True, "m": 32768, "n": 32768, "s": 512},
        # the general handle with a large sketch
        {"name": "precond_general_s1024", "kind": "precond", "psd": False, "m": 16384, "n": 16384, "s": 1024},
        # ridge regression with eight targets: three levels of iteration
        {"name": "ridge_n4096_k8", "kind": "ridge", "m": 4096, "n": 4096, "s": 512, "k": 8, "lam": 1e-2},
        # three quadrature nodes of a Schatten-1 estimate, 64 probes as one block
        {"name": "schatten_n2048", "kind": "schatten", "m": 2048, "n": 2048, "s": 256, "k": 64, "nodes": 3},
        # tall least squares, one right-hand side
        {"name": "lstsq_20000x128", "kind": "lstsq", "m": 20000, "n": 128, "s": 32, "k": 1},
        # uneven GP systems of a batch, forward and adjoint, F32 storage with FP64 refinement
        {"name": "batched_24", "kind": "batched", "systems": 24, "n_lo": 256, "n_hi": 1500, "k": 16, "a": "f32"},
        # a differentiable solve inside a training step
        {"name": "backward_n6000_k4", "kind": "backward", "n": 6000, "s": 256, "k": 4},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["path", "solve", "solve", "solve", "sketch", "sketch", "precond", "ridge", "ridge", "lstsq",
                       "schatten", "batched", "backward"])
    c = {"kind": kind}
    if kind == "path":
        n = _log_int(rng, 300, 4096)
        s = min(n // 4, _log_int(rng, 32, 256))
        c.update(n=n, s=s, k=rng.choice([1, 1, 2, 5]), outliers=max(4, s // 2))
    elif kind == "solve":
        k = rng.choice([1, 1, 3, 8, 16, 24])
        n = _log_int(rng, 2000, 20000 if k == 1 else 10000)
        c.update(n=n, s=min(n // 8, _log_int(rng, 96, 768)), k=k, a=rng.choice(["f64", "f64", "f32"]))
    elif kind == "sketch":
        a = rng.choice(["f64", "f32", "bf16"])
        c.update(m=_log_int(rng, 1000, 32768), n=_log_int(rng, 1000, 32768), a=a)
        c["s"] = min(c["n"] // 2, _log_int(rng, 48, 2048))
    elif kind == "precond":
        n = _log_int(rng, 2000, 32768)
        c.update(psd=rng.random() < 0.5, m=n, n=n, s=min(n // 8, _log_int(rng, 48, 1024)))
    elif kind == "ridge":
        n = _log_int(rng, 500, 6000)
        c.update(m=_log_int(rng, n, 2 * n), n=n, s=min(n // 4, _log_int(rng, 32, 700)),
                 k=rng.choice([1, 1, 4, 8, 13, 16, 20]), lam=10.0 ** rng.uniform(-2.0, 0.0))
    elif kind == "lstsq":
        n = _log_int(rng, 40, 128)
        c.update(m=_log_int(rng, 2000, 20000), n=n, s=max(16, n // 4), k=rng.choice([1, 1, 3]))
    elif kind == "schatten":
        n = _log_int(rng, 500, 3000)
        c.update(m=n, n=n, s=n // 8, k=rng.choice([8, 40, 64, 128]), nodes=rng.choice([2, 3, 4]))
    elif kind == "batched":
        lo = _log_int(rng, 128, 500)
        c.update(systems=rng.randint(5, 24), n_lo=lo, n_hi=min(1500, 3 * lo + 200), k=rng.choice([1, 4, 16]),
                 a=rng.choice(["f32", "f32", "f64"]))
    else:
        n = _log_int(rng, 600, 6000)
        c.update(n=n, s=min(n // 8, _log_int(rng, 64, 256)), k=rng.choice([1, 2, 4]))
    return c


# ---------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------
def _gen(seed):
    return torch.Generator(device=_DEV).manual_seed(int(seed) % (2 ** 62))


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, device=_DEV, dtype=torch.float64)


def _rbf(g, n, dim, scale, dtype):
    """The RBF kernel matrix of n Gaussian points, unit diagonal, formed in row blocks."""
    p = _randn(g, n, dim) / scale
    q = p.square().sum(1)
    A = torch.empty(n, n, dtype=dtype, device=_DEV)
    pt = p.T.contiguous()
    for i in range(0, n, 4096):
        d = (p[i:i + 4096] @ pt).mul_(2.0).sub_(q[i:i + 4096, None]).sub_(q[None, :])
        A[i:i + 4096] = d.mul_(0.5).clamp_(max=0.0).exp_()
    A.diagonal().fill_(1.0)
    # rounding of the two triangles differs in the last bits: keep one of them
    for i in range(0, n, 4096):
        e = min(n, i + 4096)
        A[i:e, e:] = A[e:, i:e].T
        B = A[i:e, i:e]
        B.copy_(torch.tril(B) + torch.tril(B, -1).T)
    return A


def _reflect(M, vs):
    """Householder reflections applied to the rows' space of M, in place."""
    for v in vs:
        M.sub_(torch.outer(v, v @ M), alpha=2.0)
    return M


def _units(g, count, n):
    v = _randn(g, count, n)
    return v / v.norm(dim=1, keepdim=True)


def _outlier_psd(g, n, outliers):
    """Q diag(e) Q^T with a few eigenvalues in 10^U(2,4) and the rest in U(0.5, 1)."""
    e = 0.5 + 0.5 * torch.rand(n, generator=g, device=_DEV, dtype=torch.float64)
    e[:outliers] = 10.0 ** (2.0 + 2.0 * torch.rand(outliers, generator=g, device=_DEV, dtype=torch.float64))
    e = torch.sort(e, descending=True).values
    Q, _ = torch.linalg.qr(_randn(g, n, n))
    A = (Q * e) @ Q.T
    return torch.tril(A) + torch.tril(A, -1).T, e


def _general(g, m, n, decay):
    """U diag(sigma) V^T, sigma_i = i^-decay, U and V products of Householder reflections."""
    sig = torch.arange(1, n + 1, device=_DEV, dtype=torch.float64) ** -decay
    A = torch.zeros(m, n, dtype=torch.float64, device=_DEV)
    A[:n, :n].diagonal().copy_(sig)
    _reflect(A, _units(g, 6, m))
    At = A.T.contiguous()
    _reflect(At, _units(g, 6, n))
    return At.T.contiguous(), sig


def _tail(eigs, s):
    """lam0 = (2/l) sum_{i>l} lambda_i with l = s/2."""
    l = max(1, s // 2)
    return float(2.0 / l * eigs[l:].sum())


def _phi(s, rows):
    return min(4 * s, rows)


def _inputs(case, seed):
    g = _gen(seed)
    kind = case["kind"]
    st = {"case": dict(case), "seed": int(seed) * 16 + 3}
    if kind == "path":
        A, e = _outlier_psd(g, case["n"], case["outliers"])
        B = _randn(g, case["k"], case["n"])
        st.update(A=A, B=B[0].clone() if case["k"] == 1 else B, lam=1e-3, lam0=_tail(e, case["s"]))
    elif kind in ("solve", "backward"):
        n = case["n"]
        A = _rbf(g, n, 8, 1.0, _DT[case.get("a", "f64")])
        B = _randn(g, case["k"], n)
        st.update(A=A, B=B[0].clone() if case["k"] == 1 else B, lam=1e-2)
    elif kind == "sketch":
        A = torch.empty(case["m"], case["n"], dtype=_DT[case["a"]], device=_DEV)
        for i in range(0, case["m"], 4096):
            A[i:i + 4096] = _randn(g, min(4096, case["m"] - i), case["n"])
        st["A"] = A
    elif kind == "precond":
        if case["psd"]:
            st.update(A=_rbf(g, case["n"], 8, 1.0, torch.float64), lam=1e-2)
        else:
            A, sig = _general(g, case["m"], case["n"], 0.75)
            st.update(A=A, lam=1e-2, lam0=_tail(sig.square(), case["s"]))
    elif kind in ("ridge", "schatten"):
        A, sig = _general(g, case["m"], case["n"], 1.0 if kind == "schatten" else 0.75)
        st.update(A=A, lam0=_tail(sig.square(), case["s"]))
        C = _randn(g, case["k"], case["n"])
        if kind == "ridge":
            st.update(B=C[0].clone() if case["k"] == 1 else C, lam=case["lam"])
        else:
            st.update(G=C)
    elif kind == "lstsq":
        m, n = case["m"], case["n"]
        sig = 1.0 + 4.0 * torch.rand(n, generator=g, device=_DEV, dtype=torch.float64)
        big = max(2, n // 32)
        sig[:big] = 10.0 ** (2.0 + torch.rand(big, generator=g, device=_DEV, dtype=torch.float64))
        sig = torch.sort(sig, descending=True).values
        U, _ = torch.linalg.qr(_randn(g, m, n))
        V, _ = torch.linalg.qr(_randn(g, n, n))
        A = ((U * sig) @ V.T).contiguous()
        B = _randn(g, case["k"], m)
        st.update(A=A, B=B[0].clone() if case["k"] == 1 else B, lam0=_tail(sig.square(), case["s"]))
    else:  # batched
        sys = []
        r = np.random.default_rng([case["systems"], case["n_lo"], case["n_hi"]])  # the sizes belong to the case
        for _ in range(case["systems"]):
            n = int(round(math.exp(r.uniform(math.log(case["n_lo"]), math.log(case["n_hi"])))))
            A = _rbf(g, n, 4, float(r.uniform(0.5, 2.0)), _DT[case["a"]])
            sys.append((A, _randn(g, case["k"], n)))
        st.update(sys=sys, lam=1e-2)
    return st


def _psd_handle(A, s, lam, seed, lam0=None):
    s = max(8, s)
    rows, signs, Y = msp.sketch(A, s, min(_GAMMA, s), seed)
    return msp.Precond("psd", rows, signs, Y, lam, lam0, _phi(s, A.shape[0]), _GAMMA, seed + 1, A=A)


def prepare(case, seed):
    st = _inputs(case, seed)
    kind = case["kind"]
    if kind in ("solve", "backward"):
        st["P"] = _psd_handle(st["A"], case["s"], st["lam"], st["seed"])
        if kind == "backward":
            st["A"].requires_grad_(True)
            st["B"].requires_grad_(True)
            st["lam_t"] = torch.tensor(st["lam"], dtype=torch.float64, device=_DEV, requires_grad=True)
    elif kind in ("precond", "ridge", "schatten"):
        psd = kind == "precond" and case["psd"]
        st["sk"] = msp.sketch(st["A"], case["s"], _GAMMA, st["seed"])
        if kind != "precond":
            st["P"] = msp.Precond("general", *st["sk"], st.get("lam", 1.0), st["lam0"], _phi(case["s"], case["m"]),
                                  _GAMMA, st["seed"] + 1)
        elif psd:
            # the handle reads the diagonal of A alone; the program still holds A
            st["lam0"] = None
    elif kind == "batched":
        st["handles"] = [_psd_handle(A, min(256, A.shape[0] // 2), st["lam"], st["seed"] + 97 * i)
                         for i, (A, _) in enumerate(st["sys"])]
    return st


# ---------------------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------------------
def run(st):
    case, kind = st["case"], st["case"]["kind"]
    if kind == "path":
        sp = msp.SketchParams(s=case["s"], gamma=_GAMMA, phi=_phi(case["s"], case["n"]), phi_gamma=_GAMMA,
                              seed=st["seed"], phi_seed=st["seed"] + 1)
        X, _, _ = msp.msp_solve(st["A"], st["B"], st["lam"], st["lam0"], sp, tol=1e-10)
        return X
    if kind == "solve":
        X, _ = msp.solve(st["P"], st["A"], st["B"], tol=1e-10, refine=1 if case["a"] != "f64" else 0)
        return X
    if kind == "sketch":
        return msp.sketch(st["A"], case["s"], _GAMMA, st["seed"])
    if kind == "precond":
        P = msp.Precond("psd" if case["psd"] else "general", *st["sk"], st["lam"], st["lam0"],
                        _phi(case["s"], case["m"]), _GAMMA, st["seed"] + 1, A=st["A"] if case["psd"] else None)
        W, Mi, M2 = P.factors()
        return {"W": W, "Mi": Mi, "M2": M2, "lam0": P.lam0}
    if kind == "ridge":
        X, _ = msp.solve(st["P"], st["A"], st["B"], normal=1, tol=1e-11)
        return X
    if kind == "lstsq":
        rows, signs, At = msp.left_sketch(st["A"], 4 * case["n"], _GAMMA, st["seed"])
        r2, s2, Y = msp.sketch(At, case["s"], _GAMMA, st["seed"] + 1)
        P = msp.Precond("general", r2, s2, Y, 0.0, st["lam0"], _phi(case["s"], At.shape[0]), _GAMMA, st["seed"] + 2)
        X, _ = msp.lstsq(P, At, st["A"], st["B"], tol=1e-11, refine_inner_tol=0.1, level3_tol=1e-6)
        return X
    if kind == "schatten":
        est, se, _ = msp.schatten(st["P"], st["A"], st["G"], p=1.0, h=_H, u_lo=_U_LO,
                                  u_hi=_U_LO + _H * (case["nodes"] - 0.5), tol=1e-11)
        return {"estimate": est, "std_err": se}
    if kind == "batched":
        sysl = [(P, A, None, B) for P, (A, B) in zip(st["handles"], st["sys"])]
        opts = {"tol": 1e-10, "refine": 1 if case["a"] != "f64" else 0}
        Xs, _ = msp.solve_batched(sysl, **opts)
        # the loss sum |X_i|^2: G = 2 X
        dB, dl, _, _ = msp.solve_batched_backward(sysl, Xs, [2.0 * x for x in Xs], **opts)
        # one tensor per kind of output: the systems' blocks one after the other
        return {"X": torch.cat([x.reshape(-1) for x in Xs]), "dB": torch.cat([x.reshape(-1) for x in dB]),
                "dlam": np.array(dl)}
    X = msp.MSPSolve.apply(st["A"], st["B"], st["lam_t"], st["P"], {"tol": 1e-10})
    dA, dB, dl = torch.autograd.grad(X.square().sum(), (st["A"], st["B"], st["lam_t"]))
    return {"X": X.detach(), "dA": dA, "dB": dB, "dlam": dl}


_H, _U_LO = 1.5, -4.0


# ---------------------------------------------------------------------------------------
# the least that a pass needs
# ---------------------------------------------------------------------------------------
def work(case):
    kind = case["kind"]
    k = case.get("k", 1)
    if kind == "path":
        n, s = case["n"], case["s"]
        return {"bytes": 8.0 * n * n / 2 + 16.0 * n * k, "flops": 2.0 * n * n * k + 2.0 * n * s * _GAMMA}
    if kind in ("solve", "backward"):
        n, s, b = case["n"], case["s"], _SIZE[case.get("a", "f64")]
        by = b * n * n / 2 + 8.0 * n * s + 16.0 * n * k
        fl = 2.0 * n * n * k + 4.0 * n * s * k
        if kind == "backward":
            by += 8.0 * n * n + 32.0 * n * k
            fl = 2 * fl + 2.0 * n * n * k
        return {"bytes": by, "flops": fl}
    if kind == "sketch":
        m, n, s, b = case["m"], case["n"], case["s"], _SIZE[case["a"]]
        return {"bytes": b * m * n + max(b, 4) * m * s + 5.0 * n * _GAMMA, "flops": 2.0 * m * n * _GAMMA}
    if kind == "precond":
        m, n, s = case["m"], case["n"], case["s"]
        f = _phi(s, m)
        by = 8.0 * m * s + 3 * 8.0 * s * s
        # the Gram product of the embedded sketch and the inverses (two for the general handle)
        fl = f * s * s + 2.0 * s ** 3 * (1 if case["psd"] else 2) + (m * s * s if case["psd"] else 0)
        return {"bytes": by, "flops": fl}
    if kind in ("ridge", "schatten"):
        m, n, s = case["m"], case["n"], case["s"]
        nd = case.get("nodes", 1)
        return {"bytes": 8.0 * m * n + 8.0 * m * s + 16.0 * n * k,
                "flops": nd * (4.0 * m * n * k + 2.0 * n * s * k) + 2.0 * m * s * s}
    if kind == "lstsq":
        m, n, s = case["m"], case["n"], case["s"]
        return {"bytes": 8.0 * m * n + 8.0 * 4 * n * n + 8.0 * (m + n) * k,
                "flops": 2.0 * m * n * _GAMMA + 4.0 * m * n * k + 2.0 * 4 * n * n * s}
    # batched: the systems' sizes are spread over the logarithm of the range
    b = _SIZE[case["a"]]
    lo, hi = case["n_lo"], case["n_hi"]
    n2 = (hi * hi - lo * lo) / (2 * math.log(hi / lo)) if hi > lo else float(lo * lo)
    return {"bytes": case["systems"] * b * n2, "flops": 2 * case["systems"] * 2.0 * n2 * k}


# ---------------------------------------------------------------------------------------
# the same results in 64 bits from dense linear algebra
# ---------------------------------------------------------------------------------------
_M64 = np.uint64(0xFFFFFFFFFFFFFFFF)
_GOLD = np.uint64(0x9E3779B97F4A7C15)


def _fmix(z):
    z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
    z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
    return z ^ (z >> np.uint64(31))


def _embedding(n, rows, gamma, seed):
    """The sparse embedding's dense (rows, n) matrix: gamma distinct rows a column, +-1/sqrt(gamma)."""
    with np.errstate(over="ignore"):
        key = _fmix(np.uint64(seed & int(_M64)) + np.arange(1, n + 1, dtype=np.uint64) * _GOLD)
        got = np.full((n, gamma), -1, dtype=np.int64)
        sign = np.ones((n, gamma))
        cnt = np.zeros(n, dtype=np.int64)
        a = 0
        while (cnt < gamma).any():
            a += 1
            u = _fmix(key + np.uint64(a) * _GOLD)
            r = (((u >> np.uint64(32)) * np.uint64(rows)) >> np.uint64(32)).astype(np.int64)
            ok = (cnt < gamma) & ~(got == r[:, None]).any(1)
            i = np.nonzero(ok)[0]
            got[i, cnt[i]] = r[i]
            sign[i, cnt[i]] = np.where(u[i] & np.uint64(1), -1.0, 1.0)
            cnt[i] += 1
    S = torch.zeros(rows, n, dtype=torch.float64, device=_DEV)
    col = torch.arange(n, device=_DEV).repeat_interleave(gamma)
    S[torch.from_numpy(got.reshape(-1)).to(_DEV), col] = torch.from_numpy(sign.reshape(-1)).to(_DEV) / math.sqrt(gamma)
    return S


def _sketch64(A, S):
    St = S.T.contiguous()
    out = torch.empty(A.shape[0], S.shape[0], dtype=torch.float64, device=_DEV)
    for i in range(0, A.shape[0], 4096):
        out[i:i + 4096] = A[i:i + 4096].double() @ St
    return out


def _spd_solve(M, B):
    """M X^T = B^T for rows of right-hand sides; two refinement steps in 64 bits."""
    L = torch.linalg.cholesky(M)
    X = torch.cholesky_solve(B.T.contiguous(), L)
    for _ in range(2):
        X = X + torch.cholesky_solve(B.T - M @ X, L)
    return X.T.contiguous()


def _shifted(A, lam):
    M = A.detach().double().clone()
    M.diagonal().add_(lam)
    return M


def _sym_inverse(M):
    M = (M + M.T) / 2
    M.diagonal().add_(1e-12 * float(M.diagonal().sum()) / M.shape[0])
    L = torch.linalg.cholesky(M)
    X = torch.cholesky_inverse(L)
    I2 = 2.0 * torch.eye(M.shape[0], dtype=M.dtype, device=M.device)
    X = X @ (I2 - M @ X)
    return (X + X.T) / 2


def exact(case, seed):
    kind = case["kind"]
    st = _inputs(case, seed)
    if kind in ("path", "solve", "backward"):
        B = st["B"]
        B2 = B if B.dim() == 2 else B[None]
        M = _shifted(st["A"], st["lam"])
        if kind != "backward":
            del st
            return _spd_solve(M, B2).reshape(B.shape)
        X = _spd_solve(M, B2)
        dB = _spd_solve(M, 2.0 * X)
        return {"X": X.reshape(B.shape), "dA": -(dB.T @ X), "dB": dB.reshape(B.shape), "dlam": -(dB * X).sum()}
    if kind == "sketch":
        return None, None, _sketch64(st["A"], _embedding(case["n"], case["s"], _GAMMA, st["seed"]))
    if kind == "precond":
        s, m, n = case["s"], case["m"], case["n"]
        S = _embedding(n, s, _GAMMA, st["seed"])
        Y = _sketch64(st["A"], S)
        F = _embedding(m, _phi(s, m), _GAMMA, st["seed"] + 1)
        Z = F @ Y
        if not case["psd"]:
            G = Z.T @ Z
            lt = st["lam"] + st["lam0"]
            return {"W": None, "Mi": _sym_inverse(G), "M2": _sym_inverse(_shifted(G, lt)), "lam0": st["lam0"]}
        W = S @ Y
        W = (W + W.T) / 2
        mu = 1e-9 * float(W.diagonal().sum()) / s
        tr = float(st["A"].diagonal().sum())
        nys = float((torch.linalg.inv(_shifted(W, mu)) * (Y.T @ Y)).sum())
        lam0 = 2.0 / (0.5 * s) * (tr - nys) if tr - nys > 1e-6 * tr else 0.0
        return {"W": W, "Mi": _sym_inverse(Z.T @ Z + (st["lam"] + lam0) * W), "M2": None, "lam0": lam0}
    if kind == "ridge":
        B = st["B"]
        M = _shifted(st["A"].T @ st["A"], st["lam"])
        return _spd_solve(M, B if B.dim() == 2 else B[None]).reshape(B.shape)
    if kind == "lstsq":
        B = st["B"]
        B2 = B if B.dim() == 2 else B[None]
        Q, R = torch.linalg.qr(st["A"])
        X = torch.linalg.solve_triangular(R, Q.T @ B2.T, upper=True)
        X = X + torch.linalg.solve_triangular(R, Q.T @ (B2.T - st["A"] @ X), upper=True)
        return X.T.reshape((B2.shape[0], case["n"]) if B.dim() == 2 else (case["n"],)).contiguous()
    if kind == "schatten":
        e, V = torch.linalg.eigh(st["A"].T @ st["A"])
        e = e.clamp_min(0.0)
        Z2 = (st["G"] @ V).square()
        vals = torch.zeros(case["k"], dtype=torch.float64, device=_DEV)
        for j in range(case["nodes"]):
            t = math.exp(_U_LO + j * _H)
            vals += _H / math.pi * math.sqrt(t) * (Z2 * (e / (e + t))).sum(1)
        return {"estimate": float(vals.mean()), "std_err": float(vals.std() / math.sqrt(case["k"]))}
    X, dB, dl = [], [], []
    for A, B in st["sys"]:
        M = _shifted(A, st["lam"])
        x = _spd_solve(M, B)
        d = _spd_solve(M, 2.0 * x)
        X.append(x.reshape(-1))
        dB.append(d.reshape(-1))
        dl.append(-float((d * x).sum()))
    return {"X": torch.cat(X), "dB": torch.cat(dB), "dlam": np.array(dl)}
