"""Timed workloads of the library's public entry points.

Every case is a dict of plain values; ``prepare`` draws its inputs on the GPU
from a seed and builds the handle a user's program would keep, ``run`` makes
one pass, ``work`` counts the bytes and flops the pass cannot do without and
``exact`` gives the same outputs from plain torch in 64 bits.

The matrices have the structure of the repository's synthetic workloads
(A = Q diag(d) Q^H with d uniform, B complex symmetric Gaussian with
||B||_2 = c min d).  Q is a product of random Householder reflectors instead
of a Haar unitary, so that a problem is drawn in milliseconds, and ||B||_2
is set by the edge 2 sqrt(m) of the Gaussian's singular values.

Eigenvectors are returned in the gauge in which the sum of their components
is real and positive.

Kinds of case:
  apply     Y = H X (``PHSolver.apply_h``)
  filter    W <- p(H^2) W, c64 or c128, one degree or one per column
            (``PHSolver.filter``)
  refined   W <- p(H^2) W by the FP64-corrected c64 filter
            (``PHSolver.filter_refined``)
  qr        Cholesky QR of a search block (``PHSolver.qr``)
  rr        oblique Rayleigh-Ritz step, back-transform and residuals
            (``PHSolver.oblique_rr``, ``PHSolver.residuals``)
  backward  eigenvalue adjoint (``PHSolver.eigval_backward``)
  solve     the nev smallest positive pairs (``PHSolver.solve``)
  tda       the nev smallest pairs of A alone (``TDASolver.solve``)
  grad      differentiable eigenvalues, forward and backward (``eigsh_ph``)
"""
import math

import numpy as np
import torch

import paper_2601_10557_amd as ph

REFLECTORS = 4


def listed():
    return [
        # one product of the Lanczos estimates on the smallest workload:
        # latency of a single call
        dict(name="apply-fp64-m500-k4", kind="apply", m=500, k=4, prec="fp64", dmin=1.0, dmax=5.0, c=0.4),
        # the whole filter step of the smallest workload: 40 dependent small
        # products
        dict(name="filter-fp64-m500-k30", kind="filter", m=500, k=30, prec="fp64", deg_lo=20, deg_hi=20, dmin=1.0,
             dmax=5.0, c=0.4),
        # first filter step of the mixed-precision solve at m = 4000
        dict(name="filter-c64-m4000-k260", kind="filter", m=4000, k=260, prec="fp32", deg_lo=20, deg_hi=20, dmin=0.5,
             dmax=10.0, c=0.3),
        # FP64 filter with a ragged size and a degree per column, some pairs
        # locked
        dict(name="filter-fp64-m2777-k145", kind="filter", m=2777, k=145, prec="fp64", deg_lo=8, deg_hi=20, dmin=0.5,
             dmax=10.0, c=0.3),
        # orthonormalisation of the full search block at m = 4000
        dict(name="qr-m4000-k520", kind="qr", m=4000, k=520, dmin=0.5, dmax=10.0, c=0.3),
        # Rayleigh-Ritz, back-transform and residuals at m = 4000 with a part
        # of the pairs locked
        dict(name="rr-m4000-k376", kind="rr", m=4000, k=376, dmin=0.5, dmax=10.0, c=0.3),
        # gradient of an eigenvalue loss at m = 4000
        dict(name="backward-m4000-nev200", kind="backward", m=4000, nev=200, dmin=0.5, dmax=10.0, c=0.3),
        # whole solve of the smallest workload, FP64
        dict(name="solve-fp64-m500", kind="solve", m=500, nev=20, nex=10, prec="fp64", tol=1e-10, passes=10.0, dmin=1.0,
             dmax=5.0, c=0.4),
        # whole mixed-precision solve on the matrices of the headline workload,
        # 120 pairs
        dict(name="solve-mixed-m4000", kind="solve", m=4000, nev=120, nex=60, prec="mixed", tol=1e-9, passes=17.0,
             dmin=0.5, dmax=10.0, c=0.3),
        # Hermitian problem on A alone
        dict(name="tda-m4000", kind="tda", m=4000, nev=120, nex=60, tol=1e-9, passes=5.0, dmin=0.5, dmax=10.0, c=0.3),
        # differentiation workload: solve and gradients with respect to A, B
        dict(name="grad-m2000", kind="grad", m=2000, nev=50, nex=20, tol=1e-12, passes=30.0, dmin=1.0, dmax=5.0,
             c=0.4),
        # one filter step of a large problem, FP64-corrected c64 products and
        # a degree per column
        dict(name="refined-m16000-k1200", kind="refined", m=16000, k=1200, deg_lo=8, deg_hi=16, dmin=1.0, dmax=20.0,
             c=0.25),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    spectrum = rng.choice([dict(dmin=1.0, dmax=5.0, c=0.4), dict(dmin=0.5, dmax=10.0, c=0.3),
                           dict(dmin=1.0, dmax=20.0, c=0.25)])
    kind = rng.choice(["apply", "filter", "filter", "refined", "qr", "rr", "backward", "solve", "tda", "grad"])
    m = _log(rng, 200, 8000)
    kmax = max(4, int(0.08 * m))
    if kind == "apply":
        return dict(kind=kind, m=m, k=_log(rng, 1, 2 * kmax), prec=rng.choice(["fp64", "fp32"]), **spectrum)
    if kind in ("filter", "refined"):
        lo = rng.randint(6, 20)
        case = dict(kind=kind, m=m, k=_log(rng, 4, kmax), deg_lo=lo, deg_hi=rng.choice([lo, rng.randint(lo, 28)]),
                    **spectrum)
        if kind == "filter":
            case["prec"] = rng.choice(["fp64", "fp32"])
        return case
    if kind in ("qr", "rr"):
        return dict(kind=kind, m=min(m, 6000), k=2 * _log(rng, 4, min(kmax, 320)), **spectrum)
    if kind == "backward":
        return dict(kind=kind, m=m, nev=_log(rng, 1, max(2, kmax // 2)), **spectrum)
    m = _log(rng, 200, 1600)
    nev = max(4, int(m * rng.uniform(0.015, 0.05)))
    nex = max(6, int(nev * rng.uniform(0.3, 0.6)))
    spectrum = rng.choice([dict(dmin=1.0, dmax=5.0, c=0.4), dict(dmin=0.5, dmax=10.0, c=0.3)])
    if kind == "solve":
        prec = rng.choice(["fp64", "mixed"])
        return dict(kind=kind, m=m, nev=nev, nex=nex, prec=prec, tol=1e-10 if prec == "fp64" else 1e-9, passes=10.0,
                    **spectrum)
    if kind == "tda":
        return dict(kind=kind, m=m, nev=nev, nex=nex, tol=1e-10, passes=5.0, **spectrum)
    return dict(kind=kind, m=m, nev=nev, nex=nex, tol=1e-11, passes=10.0, **spectrum)


# ------------------------------------------------------------------ inputs
def _cnormal(shape, gen, dtype=torch.float64):
    return torch.complex(torch.randn(shape, dtype=dtype, device="cuda", generator=gen),
                         torch.randn(shape, dtype=dtype, device="cuda", generator=gen))


def _reflect(X, us):
    """Q X for Q the product of the reflectors 1 - 2 u u^H, the last one first."""
    for u in reversed(us):
        X = X - 2.0 * u[:, None] * (u.conj()[None, :] @ X)
    return X


def _problem(case, seed):
    """(A, B, d ascending, reflectors, generator); A's eigenvector of d[i] is Q e_i."""
    m = case["m"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    d = torch.rand(m, dtype=torch.float64, device="cuda", generator=gen)
    d = torch.sort(case["dmin"] + (case["dmax"] - case["dmin"]) * d).values
    us = []
    for _ in range(REFLECTORS):
        u = _cnormal((m,), gen)
        us.append(u / torch.linalg.vector_norm(u))
    A = torch.diag(d).to(torch.complex128)
    A = _reflect(A, us)                          # Q diag(d)
    A = _reflect(A.mH.contiguous(), us)          # Q (Q diag(d))^H = Q diag(d) Q^H
    A = 0.5 * (A + A.mH)
    B = _cnormal((m, m), gen)
    B = 0.5 * (B + B.T)
    B *= case["c"] * float(d[0]) / (2.0 * math.sqrt(m))
    return A.contiguous(), B.contiguous(), d, us, gen


def _degrees(case):
    k, lo, hi = case["k"], case["deg_lo"], case["deg_hi"]
    return [lo + (hi - lo) * j // max(1, k - 1) for j in range(k)]


def _mu(case, d, k):
    """Filter interval as the spectral estimates give it: near the smallest and
    largest eigenvalue and at the one after the search block."""
    return 0.95 * case["dmin"], float(d[min(k, d.numel() - 1)]), 1.02 * case["dmax"]


def _search_block(case, d, us, gen, k):
    """n x k block close to the eigenvectors of the k smallest values: the
    unit vectors [Q e_i; 0] with 2% of noise."""
    m = case["m"]
    E = torch.zeros((m, k), dtype=torch.complex128, device="cuda")
    E[torch.arange(k), torch.arange(k)] = 1.0
    W = torch.cat([_reflect(E, us), torch.zeros_like(E)])
    return W + (0.02 / math.sqrt(2 * m)) * _cnormal((2 * m, k), gen)


def _k_conj(W):
    m = W.shape[0] // 2
    return torch.cat([W[m:], W[:m]]).conj()


def prepare(case, seed):
    A, B, d, us, gen = _problem(case, seed)
    kind, m = case["kind"], case["m"]
    st = dict(case=case, A=A, B=B)
    if kind == "apply":
        k = case["k"]
        st["solver"] = ph.PHSolver(A, B, 8, 8, precision=ph.MIXED if case["prec"] == "fp32" else ph.FP64)
        X = _cnormal((2 * m, k), gen)
        st["X"] = ph.colmajor(X.to(torch.complex64) if case["prec"] == "fp32" else X)
    elif kind == "filter":
        k = case["k"]
        st["solver"] = ph.PHSolver(A, B, k, 0, precision=ph.MIXED if case["prec"] == "fp32" else ph.FP64)
        W = _cnormal((2 * m, k), gen)
        st["W"] = ph.colmajor(W.to(torch.complex64) if case["prec"] == "fp32" else W)
        st["mu"], st["degs"] = _mu(case, d, k), _degrees(case)
    elif kind == "refined":
        k = case["k"]
        st["solver"] = ph.PHSolver(A, B, k, 0, precision=ph.MIXED)
        W = _search_block(case, d, us, gen, k)
        W = W / torch.linalg.vector_norm(W, dim=0)
        lam = d[:k].clone()
        st["R"] = ph.colmajor(_h(A, B, W) - W * lam)
        st["W"] = ph.colmajor(W)
        st["lam"] = lam.cpu().numpy()
        st["mu"], st["degs"] = _mu(case, d, k), _degrees(case)
    elif kind in ("qr", "rr"):
        k = case["k"]
        st["solver"] = ph.PHSolver(A, B, k // 2, 0)
        W = _search_block(case, d, us, gen, k // 2)
        X = torch.cat([W, _k_conj(W)], dim=1)
        if kind == "rr":
            # Cholesky QR twice: orthonormal to rounding, the block is well conditioned
            for _ in range(2):
                L = torch.linalg.cholesky((X.mH @ X).cpu())
                X = X @ torch.linalg.inv(L).mH.contiguous().cuda()
        st["X"] = ph.colmajor(X)
    elif kind == "backward":
        nev = case["nev"]
        st["solver"] = ph.PHSolver(A, B, nev, 0)
        V = _search_block(case, d, us, gen, nev)
        st["V"] = ph.colmajor(V / torch.linalg.vector_norm(V, dim=0))
        st["g"] = torch.randn(nev, dtype=torch.float64, device="cuda", generator=gen).cpu().numpy()
    elif kind in ("solve", "grad"):
        nev, nex = case["nev"], case["nex"]
        st["W0"] = ph.colmajor(_cnormal((2 * m, nev + nex), gen))
        st["Lz"] = ph.colmajor(_cnormal((2 * m, 4), gen))
        if kind == "solve":
            st["solver"] = ph.PHSolver(A, B, nev, nex, deg=20, tol=case["tol"], max_iter=100,
                                       precision=ph.MIXED if case["prec"] == "mixed" else ph.FP64)
        else:
            st["w"] = torch.randn(nev, dtype=torch.float64, device="cuda", generator=gen)
    elif kind == "tda":
        nev, nex = case["nev"], case["nex"]
        st["W0"] = ph.colmajor(_cnormal((m, nev + nex), gen))
        st["Lz"] = ph.colmajor(_cnormal((m, 4), gen))
        st["solver"] = ph.TDASolver(A, nev, nex, deg=20, tol=case["tol"], max_iter=100)
    else:
        raise ValueError(kind)
    return st


# -------------------------------------------------------------------- pass
def _gauge(V):
    s = V.sum(dim=0)
    return V * (s.conj() / s.abs())


def run(state):
    case, kind, s = state["case"], state["case"]["kind"], state.get("solver")
    if kind == "apply":
        return s.apply_h(state["X"], prec=ph.FP32 if case["prec"] == "fp32" else ph.FP64)
    if kind == "filter":
        return s.filter(state["W"].clone(), *state["mu"], degs=state["degs"],
                        prec=ph.FP32 if case["prec"] == "fp32" else ph.FP64)
    if kind == "refined":
        return s.filter_refined(state["W"].clone(), state["R"], state["lam"], *state["mu"], degs=state["degs"])
    if kind == "qr":
        Q = state["X"].clone()
        R, _ = s.qr(Q)
        return dict(Q=Q, R=R)
    if kind == "rr":
        ritz, Z, T = s.oblique_rr(state["X"])
        V, res = s.residuals(state["X"], T, Z, ritz)
        return dict(ritz=ritz, T=T, V=_gauge(V), res=res)
    if kind == "backward":
        GA, GB = s.eigval_backward(state["V"], state["g"])
        return dict(GA=GA, GB=GB)
    if kind in ("solve", "tda"):
        ev, V, _, _ = s.solve(state["W0"], state["Lz"])
        return dict(ev=ev, V=_gauge(V))
    A, B = state["A"].detach().requires_grad_(True), state["B"].detach().requires_grad_(True)
    lam = ph.eigsh_ph(A, B, case["nev"], case["nex"], state["W0"], state["Lz"], deg=20, tol=case["tol"], max_iter=100)
    (lam * state["w"]).sum().backward()
    return dict(lam=lam.detach(), GA=A.grad, GB=B.grad)


def work(case):
    kind, m = case["kind"], case["m"]
    n = 2 * m
    ab = 2.0 * 16 * m * m                      # A and B, read once
    hx = 4.0 * n * n                           # real flops of H x (half on K-real columns)
    if kind == "apply":
        elem = 8 if case["prec"] == "fp32" else 16
        return dict(bytes=ab + 2.0 * n * case["k"] * elem, flops=hx * case["k"])
    if kind in ("filter", "refined"):
        elem = 8 if case.get("prec") == "fp32" else 16
        return dict(bytes=ab + (3.0 if kind == "refined" else 2.0) * n * case["k"] * elem,
                    flops=2.0 * hx * sum(_degrees(case)))
    if kind == "qr":
        k = case["k"]
        # two passes of a Hermitian Gram matrix and a triangular product
        return dict(bytes=2.0 * 16 * n * k + 16.0 * k * k, flops=2 * 8.0 * n * k * k)
    if kind == "rr":
        k = case["k"]
        # H Q, the two Hermitian k x k quotients, Q Z and T Z on half the columns
        return dict(bytes=ab + 16.0 * n * (2 * k + k / 2),
                    flops=hx * k + 4.0 * n * k * k + 2.0 * n * k * k + 8.0 * n * k * k + 32.0 * k ** 3)
    if kind == "backward":
        return dict(bytes=ab + 16.0 * n * case["nev"], flops=16.0 * m * m * case["nev"])
    nev, nex = case["nev"], case["nex"]
    nevex = nev + nex
    if kind == "tda":
        return dict(bytes=0.5 * ab + 16.0 * m * (nevex + nev), flops=case["passes"] * 20 * 0.5 * hx * nevex)
    out = dict(bytes=ab + 16.0 * n * (nevex + nev), flops=case["passes"] * 40 * hx * nevex)
    if kind == "grad":
        out["bytes"] += ab
        out["flops"] += 16.0 * m * m * nev
    return out


# ------------------------------------------------------------- 64-bit values
def _h(A, B, X):
    m = A.shape[0]
    x, y = X[:m], X[m:]
    return torch.cat([A @ x + B @ y, -(B @ x.conj() + A @ y.conj()).conj()])


def _exact_filter(A, B, W, mu, degs):
    mu1, mu_nevex, mu_n = mu
    c, e = 0.5 * (mu_n ** 2 + mu_nevex ** 2), 0.5 * (mu_n ** 2 - mu_nevex ** 2)
    s1 = e / (mu1 ** 2 - c)
    degs = torch.tensor(degs, device=W.device)
    out = W.clone()
    prev, cur, sigma = W, (s1 / e) * (_h(A, B, _h(A, B, W)) - c * W), s1
    for s in range(1, int(degs.max()) + 1):
        out[:, degs == s] = cur[:, degs == s]
        nxt = 1.0 / (2.0 / s1 - sigma)
        prev, cur = cur, (2.0 * nxt / e) * (_h(A, B, _h(A, B, cur)) - c * cur) - sigma * nxt * prev
        sigma = nxt
    return out


def _exact_pairs(A, B, nev):
    """The nev smallest positive eigenpairs of H, from the Hermitian problem
    L^H S L of the positive definite S H = L L^H."""
    m = A.shape[0]
    A, B = A.cpu().numpy(), B.cpu().numpy()
    L = np.linalg.cholesky(np.block([[A, B], [B.conj(), A.conj()]]))
    SL = L.copy()
    SL[m:] *= -1.0
    th, Y = np.linalg.eigh(L.conj().T @ SL)      # values lambda of H, vectors S L y
    lam, V = th[m:m + nev], SL @ Y[:, m:m + nev]
    return lam, torch.from_numpy(V / np.linalg.norm(V, axis=0))


def _adjoint(V, g):
    m = V.shape[0] // 2
    x, y = V[:m], V[m:]
    gt = g / (x.abs().square().sum(0) - y.abs().square().sum(0))
    GA = (x * gt) @ x.mH + (y.conj() * gt) @ y.T
    GB = (x * gt) @ y.mH + (y.conj() * gt) @ x.T
    return GA, GB


def exact(case, seed):
    kind, m = case["kind"], case["m"]
    if kind in ("solve", "grad") and m > 1000:
        return None                               # the dense eigenproblem takes too long
    if kind == "tda":
        _, _, d, us, _ = _problem(case, seed)
        nev = case["nev"]
        E = torch.zeros((m, nev), dtype=torch.complex128, device="cuda")
        E[torch.arange(nev), torch.arange(nev)] = 1.0
        return dict(ev=d[:nev], V=_gauge(_reflect(E, us)))
    st = prepare(case, seed)
    A, B = st["A"], st["B"]
    if kind == "apply":
        return _h(A, B, st["X"].to(torch.complex128))
    if kind in ("filter", "refined"):
        return _exact_filter(A, B, st["W"].to(torch.complex128), st["mu"], st["degs"])
    if kind == "qr":
        Q, R = torch.linalg.qr(st["X"].cpu())
        p = torch.diagonal(R) / torch.diagonal(R).abs()
        return dict(Q=Q * p, R=R * p.conj()[:, None])
    if kind == "rr":
        Q = st["X"]
        T = _h(A, B, Q)
        M = (Q[:m].mH @ T[:m] - Q[m:].mH @ T[m:]).cpu()
        N = (Q[:m].mH @ Q[:m] - Q[m:].mH @ Q[m:]).cpu()
        L = torch.linalg.cholesky(0.5 * (M + M.mH))
        Li = torch.linalg.inv(L)
        G = Li @ N @ Li.mH.contiguous()
        th, Y = torch.linalg.eigh(0.5 * (G + G.mH))
        k2 = Q.shape[1] // 2
        lam = 1.0 / th.flip(0)[:k2]
        Z = (Li.mH.contiguous() @ Y.flip(1)[:, :k2]).cuda()
        V, TZ = Q @ Z, T @ Z
        nu = torch.linalg.vector_norm(V, dim=0)
        res = torch.linalg.vector_norm(TZ - V * lam.cuda(), dim=0) / nu
        return dict(ritz=lam, T=T, V=_gauge(V / nu), res=res)
    if kind == "backward":
        GA, GB = _adjoint(st["V"], torch.from_numpy(st["g"]).cuda())
        return dict(GA=GA, GB=GB)
    if kind == "solve":
        lam, V = _exact_pairs(A, B, case["nev"])
        return dict(ev=lam, V=_gauge(V))
    lam, V = _exact_pairs(A, B, case["nev"])
    GA, GB = _adjoint(V, st["w"].cpu())
    return dict(lam=torch.from_numpy(lam), GA=GA, GB=GB)
