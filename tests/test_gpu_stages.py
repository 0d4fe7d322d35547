"""GPU parity of each stage of the C ABI against the CPU oracle.

Sizes span several kernel tiles with ragged tails (m = 300: 128-row tiles
end at 44 rows; 2k = 74 output columns end mid-tile).  Tolerances:
FP64 stages ~1e-12 relative (rounding of an O(n) inner product), c64
stages 1e-5 relative (unit roundoff 6e-8 times the inner-product length).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from oracle import chebyshev, dense, hamiltonian as ham, qr as oqr, rayleigh_ritz, residuals as ores, solver as osolver
from paper_2601_10557_amd import FP32, FP64, ChasePHError, PHSolver, empty_cm
from paper_2601_10557_amd import _lib
from synth import make_problem, complex_normal
from gpu_helpers import align_columns, dev_blocks, print_case, to_dev, to_host
from cases import decoupled_singular_case


def problem(m=300, seed=0, coupling=0.4, nev=12, nex=8):
    return make_problem(m, lambda rng, mm: rng.uniform(1.0, 5.0, mm), coupling, nev, nex, 10, 1e-10, seed=seed)


@pytest.fixture(scope="module")
def prob():
    return problem()


@pytest.fixture(scope="module")
def solver(prob):
    A, B = dev_blocks(prob)
    return PHSolver(A, B, prob.nev, prob.nex)


@pytest.mark.parametrize("k", [1, 5, 37])
def test_apply_h_fp64(prob, solver, k):
    print_case("apply_h_fp64", m=prob.m, k=k)
    rng = np.random.default_rng(k)
    X = complex_normal(rng, (prob.n, k))
    Y = to_host(solver.apply_h(to_dev(X)))
    ref = ham.apply_h(prob.A, prob.B, X)
    assert np.max(np.abs(Y - ref)) <= 1e-12 * np.max(np.abs(ref))


def test_apply_h_empty(solver):
    X = empty_cm(solver.n, 0)
    Y = solver.apply_h(X)
    assert Y.shape == (solver.n, 0)


@pytest.mark.parametrize("k", [3, 37])
def test_apply_h_fp32(prob, solver, k):
    print_case("apply_h_fp32", m=prob.m, k=k)
    rng = np.random.default_rng(100 + k)
    X = complex_normal(rng, (prob.n, k))
    Y = to_host(solver.apply_h(to_dev(X, torch.complex64), prec=FP32)).astype(np.complex128)
    ref = ham.apply_h(prob.A, prob.B, X.astype(np.complex64).astype(np.complex128))
    assert np.max(np.abs(Y - ref)) <= 1e-5 * np.max(np.abs(ref))


# every c64 tile shape of the real H X GEMM (0: 256 x 128, 1: 256 x 64 on
# the 32x32x2 MFMA, 2: 256 x 32 on the 16x16x4 MFMA), with and without the
# split-K reduction; "cfg,splits" forces the plan of each launch
@pytest.mark.parametrize("plan", ["0,1", "0,4", "0,9", "1,1", "1,5", "2,1", "2,3", "2,8"])
@pytest.mark.parametrize("k", [37, 61])
def test_apply_h_fp32_every_tile_plan(prob, solver, plan, k, monkeypatch):
    print_case("apply_h_fp32_plan", m=prob.m, k=k, plan=plan)
    monkeypatch.setenv("CHASE_PH_APPLY_PLAN", plan)
    rng = np.random.default_rng(200 + k)
    X = complex_normal(rng, (prob.n, k))
    Y = to_host(solver.apply_h(to_dev(X, torch.complex64), prec=FP32)).astype(np.complex128)
    ref = ham.apply_h(prob.A, prob.B, X.astype(np.complex64).astype(np.complex128))
    assert np.max(np.abs(Y - ref)) <= 1e-5 * np.max(np.abs(ref))


@pytest.mark.parametrize("k", [1, 37, 70])
def test_apply_h_fp64_kreal(prob, solver80, k):
    # K-real columns x = [a; conj(a)]: H x = [t; -conj(t)] from half the
    # products, against the oracle's H X and the general c128 mode
    print_case("apply_h_fp64_kreal", m=prob.m, k=k)
    rng = np.random.default_rng(500 + k)
    a = complex_normal(rng, (prob.m, k))
    X = np.concatenate([a, a.conj()], axis=0)
    Y = to_host(solver80.apply_h(to_dev(X), prec=_lib.FP64_KREAL))
    ref = ham.apply_h(prob.A, prob.B, X)
    assert np.max(np.abs(Y - ref)) <= 1e-12 * np.max(np.abs(ref))
    Yg = to_host(solver80.apply_h(to_dev(X), prec=FP64))
    assert np.max(np.abs(Y - Yg)) <= 1e-13 * np.max(np.abs(ref))


# every c128 tile width ("w,parts": tiles of at most 8 >> w fragments of 16
# columns, about so many parts of K each)
@pytest.mark.parametrize("plan", ["0,1", "0,3", "1,1", "1,4", "2,1", "2,6"])
@pytest.mark.parametrize("k", [37, 61])
def test_apply_h_fp64_every_tile_plan(prob, solver, plan, k, monkeypatch):
    print_case("apply_h_fp64_plan", m=prob.m, k=k, plan=plan)
    monkeypatch.setenv("CHASE_PH_APPLY_PLAN", plan)
    rng = np.random.default_rng(300 + k)
    X = complex_normal(rng, (prob.n, k))
    Y = to_host(solver.apply_h(to_dev(X)))
    ref = ham.apply_h(prob.A, prob.B, X)
    assert np.max(np.abs(Y - ref)) <= 1e-12 * np.max(np.abs(ref))


# K-real columns a few past a multiple of 128 (1 to 33 of them) and of 64: the last
# tile has few of its columns
@pytest.mark.parametrize("k,plan", [(129, "0,1"), (130, "0,3"), (161, "0,1"), (129, "1,1"), (129, "1,4")])
def test_apply_h_fp64_kreal_short_last_tile(prob, solver80, k, plan, monkeypatch):
    print_case("apply_h_fp64_kreal_short_tile", m=prob.m, k=k, plan=plan)
    monkeypatch.setenv("CHASE_PH_APPLY_PLAN", plan)
    rng = np.random.default_rng(600 + k)
    a = complex_normal(rng, (prob.m, k))
    X = np.concatenate([a, a.conj()], axis=0)
    Y = to_host(solver80.apply_h(to_dev(X), prec=_lib.FP64_KREAL))
    ref = ham.apply_h(prob.A, prob.B, X)
    assert np.max(np.abs(Y - ref)) <= 1e-12 * np.max(np.abs(ref))


# 2k a few columns past a multiple of 128 (k % 64 <= 20; k >= 64): the
# library splits the launch by columns, in one launch (c64 with 64 < k <= 80:
# one column of wide tiles instead)
@pytest.mark.parametrize("k", [73, 84, 132, 145, 260])
def test_apply_h_column_split(prob, solver, k):
    print_case("apply_h_column_split", m=prob.m, k=k)
    rng = np.random.default_rng(400 + k)
    X = complex_normal(rng, (prob.n, k))
    Y64 = to_host(solver.apply_h(to_dev(X)))
    ref = ham.apply_h(prob.A, prob.B, X)
    assert np.max(np.abs(Y64 - ref)) <= 1e-12 * np.max(np.abs(ref))
    Y32 = to_host(solver.apply_h(to_dev(X, torch.complex64), prec=FP32)).astype(np.complex128)
    ref32 = ham.apply_h(prob.A, prob.B, X.astype(np.complex64).astype(np.complex128))
    assert np.max(np.abs(Y32 - ref32)) <= 1e-5 * np.max(np.abs(ref32))


# c64 products with 64 < k <= 80 on one column of wide tiles (256 x 160): 2k
# up to exactly the tile width (k = 80) and ragged (k = 65, 73); k = 81 and
# k = 132 take the split launch beside them
@pytest.mark.parametrize("k", [65, 73, 80, 81, 132])
def test_apply_h_fp32_wide_last_column(prob, solver, k):
    print_case("apply_h_fp32_wide", m=prob.m, k=k)
    rng = np.random.default_rng(450 + k)
    X = complex_normal(rng, (prob.n, k))
    Y32 = to_host(solver.apply_h(to_dev(X, torch.complex64), prec=FP32)).astype(np.complex128)
    ref32 = ham.apply_h(prob.A, prob.B, X.astype(np.complex64).astype(np.complex128))
    assert np.max(np.abs(Y32 - ref32)) <= 1e-5 * np.max(np.abs(ref32))


# the c64 split launch with every main tile shape (the remainder keeps the
# narrow one): one pair kernel per main shape, or two plain launches when
# the main part is on the narrow shape too; c128 products on the same plans
@pytest.mark.parametrize("plan", ["0,1", "0,3", "1,2", "2,4"])
@pytest.mark.parametrize("k", [73, 145])
def test_apply_h_column_split_every_main_plan(prob, solver, plan, k, monkeypatch):
    print_case("apply_h_column_split_plan", m=prob.m, k=k, plan=plan)
    monkeypatch.setenv("CHASE_PH_APPLY_PLAN", plan)
    rng = np.random.default_rng(500 + k)
    X = complex_normal(rng, (prob.n, k))
    Y64 = to_host(solver.apply_h(to_dev(X)))
    ref = ham.apply_h(prob.A, prob.B, X)
    assert np.max(np.abs(Y64 - ref)) <= 1e-12 * np.max(np.abs(ref))
    Y32 = to_host(solver.apply_h(to_dev(X, torch.complex64), prec=FP32)).astype(np.complex128)
    ref32 = ham.apply_h(prob.A, prob.B, X.astype(np.complex64).astype(np.complex128))
    assert np.max(np.abs(Y32 - ref32)) <= 1e-5 * np.max(np.abs(ref32))


def test_apply_h_more_columns_than_the_packed_buffer(prob, solver):
    # the packed operand holds 512 columns: k = 530 runs as 512 + 18
    print_case("apply_h_chunks", m=prob.m, k=530)
    rng = np.random.default_rng(530)
    X = complex_normal(rng, (prob.n, 530))
    Y = to_host(solver.apply_h(to_dev(X)))
    ref = ham.apply_h(prob.A, prob.B, X)
    assert np.max(np.abs(Y - ref)) <= 1e-12 * np.max(np.abs(ref))


def _mus(prob):
    lam, _ = dense.dense_ph_eig(prob.A, prob.B)
    return 0.95 * lam[0], lam[prob.nevex - 1], 1.02 * lam[-1]


@pytest.mark.parametrize("degs", [[1] * 6, [4] * 7, [7] * 5, [1, 2, 2, 3, 7, 7, 10, 11]])
def test_filter_fp64(prob, solver, degs):
    print_case("filter_fp64", m=prob.m, degs=degs)
    mu1, mu_nevex, mu_n = _mus(prob)
    rng = np.random.default_rng(len(degs) + sum(degs))
    W = osolver.init_block(complex_normal(rng, (prob.n, len(degs))), 1e-3)
    Wd = to_dev(W)
    solver.filter(Wd, mu1, mu_nevex, mu_n, degs=degs, prec=FP64)
    ref = chebyshev.chebyshev_filter(prob.A, prob.B, W, np.array(degs), mu1, mu_nevex, mu_n)
    got = to_host(Wd)
    err = np.linalg.norm(got - ref, axis=0) / np.linalg.norm(ref, axis=0)
    assert np.max(err) < 1e-11, err


def test_filter_fp64_column_split(prob):
    # 132 columns: every product of the recurrence takes the column split
    print_case("filter_fp64_column_split", m=prob.m, k=132)
    A, B = dev_blocks(prob)
    wide = PHSolver(A, B, 100, 40)
    mu1, mu_nevex, mu_n = _mus(prob)
    rng = np.random.default_rng(7)
    W = osolver.init_block(complex_normal(rng, (prob.n, 132)), 1e-3)
    Wd = to_dev(W)
    degs = [3] * 132
    wide.filter(Wd, mu1, mu_nevex, mu_n, degs=degs, prec=FP64)
    wide.close()
    ref = chebyshev.chebyshev_filter(prob.A, prob.B, W, np.array(degs), mu1, mu_nevex, mu_n)
    err = np.linalg.norm(to_host(Wd) - ref, axis=0) / np.linalg.norm(ref, axis=0)
    assert np.max(err) < 1e-11, err


def test_filter_fp32(prob, solver):
    print_case("filter_fp32", m=prob.m)
    mu1, mu_nevex, mu_n = _mus(prob)
    rng = np.random.default_rng(7)
    degs = [2, 5, 5, 9, 12]
    W = osolver.init_block(complex_normal(rng, (prob.n, len(degs))), 1e-3)
    Wd = to_dev(W, torch.complex64)
    solver.filter(Wd, mu1, mu_nevex, mu_n, degs=degs, prec=FP32)
    ref = chebyshev.chebyshev_filter(prob.A, prob.B, W, np.array(degs), mu1, mu_nevex, mu_n)
    got = to_host(Wd).astype(np.complex128)
    err = np.linalg.norm(got - ref, axis=0) / np.linalg.norm(ref, axis=0)
    assert np.max(err) < 1e-4, err


@pytest.mark.parametrize("eps", [1e-2, 1e-5, 1e-8])
def test_filter_refined_accuracy_tracks_the_residual(prob, solver, eps):
    # c64 products + FP64 refinement: the error is relative to the
    # correction term, so near-eigenvectors are filtered to FP64 accuracy
    # while the plain c64 filter stays at ~1e-6 relative.
    print_case("filter_refined", m=prob.m, eps=eps)
    lam, Vp = dense.dense_ph_eig(prob.A, prob.B)
    mu1, mu_nevex, mu_n = _mus(prob)
    rng = np.random.default_rng(11)
    k = 6
    V = Vp[:, :k] + eps * complex_normal(rng, (prob.n, k))
    V = V / np.linalg.norm(V, axis=0)[None, :]
    HV = ham.apply_h(prob.A, prob.B, V)
    lr = np.real(np.einsum("ij,ij->j", V.conj(), HV))
    R = HV - V * lr[None, :]
    degs = [2, 5, 5, 8, 12, 12]
    ref = chebyshev.chebyshev_filter(prob.A, prob.B, V, np.array(degs), mu1, mu_nevex, mu_n)
    Wd = to_dev(V)
    solver.filter_refined(Wd, to_dev(R), lr, mu1, mu_nevex, mu_n, degs=degs)
    got = to_host(Wd)
    err = np.linalg.norm(got - ref, axis=0) / np.linalg.norm(ref, axis=0)
    assert np.max(err) < 1e-3 * eps + 1e-12, err


def test_filter_kconj_equivariance(prob, solver):
    # Thm 4.2 on the device path
    mu1, mu_nevex, mu_n = _mus(prob)
    rng = np.random.default_rng(3)
    W = complex_normal(rng, (prob.n, 4))
    a = to_dev(W)
    b = to_dev(ham.apply_k_conj(W))
    solver.filter(a, mu1, mu_nevex, mu_n, degs=[6] * 4)
    solver.filter(b, mu1, mu_nevex, mu_n, degs=[6] * 4)
    x, y = to_host(a), to_host(b)
    assert np.max(np.abs(ham.apply_k_conj(x) - y)) <= 1e-11 * np.max(np.abs(y))


def _search_block(prob, kh, seed=0):
    rng = np.random.default_rng(seed)
    mu1, mu_nevex, mu_n = _mus(prob)
    W = osolver.init_block(complex_normal(rng, (prob.n, kh)), 1e-3)
    W = chebyshev.chebyshev_filter(prob.A, prob.B, W, 6, mu1, mu_nevex, mu_n)
    return np.concatenate([W, ham.apply_k_conj(W)], axis=1)


@pytest.mark.parametrize("kh", [3, 20])
def test_qr(prob, solver, kh):
    print_case("qr", m=prob.m, k=2 * kh)
    X = _search_block(prob, kh)
    Xd = to_dev(X)
    R, shifted = solver.qr(Xd)
    Q, R = to_host(Xd), to_host(R)
    Qr, Rr, sh = oqr.cholqr2(X)
    assert not shifted and not sh
    k = X.shape[1]
    assert np.max(np.abs(Q.conj().T @ Q - np.eye(k))) < 1e-12
    assert np.max(np.abs(Q @ R - X)) < 1e-12 * np.max(np.abs(X))
    assert np.max(np.abs(np.tril(R, -1))) == 0.0
    assert np.allclose(np.diag(R).imag, 0) and np.all(np.diag(R).real > 0)
    assert np.max(np.abs(Q - Qr)) < 1e-9
    assert np.max(np.abs(R - Rr)) < 1e-9 * np.max(np.abs(Rr))


def test_qr_shifted_fallback(solver, prob):
    print_case("qr_shifted", m=prob.m)
    rng = np.random.default_rng(1)
    n, k = prob.n, 24
    U, _ = np.linalg.qr(complex_normal(rng, (n, k)))
    Vh, _ = np.linalg.qr(complex_normal(rng, (k, k)))
    X = (U * np.logspace(0, -13, k)[None, :]) @ Vh.conj().T
    Xd = to_dev(X)
    R, shifted = solver.qr(Xd)
    Q, R = to_host(Xd), to_host(R)
    assert shifted == 1
    assert np.max(np.abs(Q.conj().T @ Q - np.eye(k))) < 1e-12
    assert np.max(np.abs(Q @ R - X)) < 1e-12


@pytest.fixture(scope="module")
def solver80(prob):
    """Handle with nevex = 40: QR blocks of up to 80 columns."""
    A, B = dev_blocks(prob)
    return PHSolver(A, B, 20, 20)


def test_qr_householder_fallback_unique_part(solver80, prob):
    # zero last column: both Cholesky variants break down, and the leading
    # 69 columns of the Householder QR are the unique QR (three panels, the
    # last one ragged)
    print_case("qr_householder_unique", m=prob.m, k=70)
    rng = np.random.default_rng(31)
    X = complex_normal(rng, (prob.n, 70))
    X[:, 69] = 0
    Xd = to_dev(X)
    R, variant = solver80.qr(Xd)
    Q, R = to_host(Xd), to_host(R)
    Qo, Ro, vo = oqr.orthonormalise(X)
    assert variant == 2 and vo == 2
    assert np.max(np.abs(Q.conj().T @ Q - np.eye(70))) < 1e-12
    assert np.max(np.abs(Q @ R - X)) < 1e-12 * np.max(np.abs(X))
    assert np.max(np.abs(np.tril(R, -1))) == 0.0
    d = np.diag(R)
    assert np.all(d.imag == 0) and np.all(d.real >= 0)
    assert d[69] == 0
    assert np.max(np.abs(Q[:, :69] - Qo[:, :69])) < 1e-11
    assert np.max(np.abs(R[:69, :] - Ro[:69, :])) < 1e-11 * np.max(np.abs(Ro))


def test_qr_householder_fallback_rank_deficient(solver80, prob):
    # a zero column in the first panel and a repeated one in the second
    # (k = 45: a full panel of 32 and a ragged one of 13)
    print_case("qr_householder_deficient", m=prob.m, k=45)
    rng = np.random.default_rng(32)
    X = complex_normal(rng, (prob.n, 45))
    X[:, 3] = 0
    X[:, 40] = X[:, 7]
    Xd = to_dev(X)
    R, variant = solver80.qr(Xd)
    Q, R = to_host(Xd), to_host(R)
    Qo, _, vo = oqr.orthonormalise(X)
    assert variant == 2 and vo == 2
    assert np.max(np.abs(Q.conj().T @ Q - np.eye(45))) < 1e-12
    assert np.max(np.abs(Q @ R - X)) < 1e-12 * np.max(np.abs(X))
    d = np.diag(R)
    assert np.all(d.imag == 0) and np.all(d.real >= 0)
    assert d[3] == 0 and abs(d[40]) < 1e-12 * np.max(np.abs(X))
    assert np.all(np.delete(d.real, [3, 40]) > 1e-3 * np.max(np.abs(X)))
    assert np.max(np.abs(Q[:, :3] - Qo[:, :3])) < 1e-12


def test_qr_many_cholesky_blocks(prob, solver260):
    # k = 260: the Gram matrix is padded to 320, five 64-column blocks of the
    # blocked Cholesky (diagonal-block factor and inverse, panel, update) and
    # of the blocked inverse; Q and R are unique, so they match the oracle's
    print_case("qr_many_blocks", m=prob.m, k=260)
    rng = np.random.default_rng(41)
    X = complex_normal(rng, (prob.n, 260))
    Xd = to_dev(X)
    R, shifted = solver260.qr(Xd)
    Q, R = to_host(Xd), to_host(R)
    Qr, Rr, sh = oqr.cholqr2(X)
    assert not shifted and not sh
    assert np.max(np.abs(Q.conj().T @ Q - np.eye(260))) < 1e-12
    assert np.max(np.abs(Q @ R - X)) < 1e-12 * np.max(np.abs(X))
    assert np.max(np.abs(np.tril(R, -1))) == 0.0
    assert np.allclose(np.diag(R).imag, 0) and np.all(np.diag(R).real > 0)
    assert np.max(np.abs(Q - Qr)) < 1e-10
    assert np.max(np.abs(R - Rr)) < 1e-10 * np.max(np.abs(Rr))


@pytest.mark.parametrize("kh", [2, 20])
def test_oblique_rr_and_residuals(prob, solver, kh):
    print_case("oblique_rr", m=prob.m, k=2 * kh)
    X = _search_block(prob, kh, seed=5)
    Q, _, _ = oqr.cholqr2(X)
    lam_ref, Z_ref, T_ref = rayleigh_ritz.oblique_rr(prob.A, prob.B, Q)
    Qd = to_dev(Q)
    ritz, Z, T = solver.oblique_rr(Qd)
    assert np.allclose(ritz, lam_ref, rtol=1e-11, atol=0)
    assert np.max(np.abs(to_host(T) - T_ref)) < 1e-12 * np.max(np.abs(T_ref))
    Vref = ores.back_transform(Q, Z_ref)
    rref = ores.residual_norms(prob.A, prob.B, Vref, lam_ref)
    V, res = solver.residuals(Qd, T, Z, ritz)
    V = align_columns(to_host(V), Vref)
    assert np.max(np.abs(V - Vref)) < 1e-8
    assert np.allclose(res, rref, rtol=1e-6, atol=1e-12)
    # Thm 4.5 consequence: the positive Ritz pairs satisfy the Galerkin
    # condition with the dual basis S Q
    Vh = to_host(solver.residuals(Qd, T, Z, ritz)[0])
    R = ham.apply_h(prob.A, prob.B, Vh) - Vh * ritz[None, :]
    assert np.max(np.abs(Q.conj().T @ ham.apply_s(R))) < 1e-11


def test_rr_exact_invariant_subspace(prob, solver):
    lam, Vp = dense.dense_ph_eig(prob.A, prob.B)
    X = np.concatenate([Vp[:, :6], ham.apply_k_conj(Vp[:, :6])], axis=1)
    Q, _, _ = oqr.cholqr2(X)
    ritz, Z, T = solver.oblique_rr(to_dev(Q))
    assert np.allclose(ritz, lam[:6], rtol=1e-12)


def test_rr_reports_an_unconverged_jacobi_eigensolver(prob):
    # one sweep cannot diagonalise the quotient of a random block:
    # CHASE_PH_ERR_EIG, not a silently inaccurate result; with the default
    # limit the same call succeeds
    print_case("rr_jacobi_sweep_limit", m=prob.m, k=40)
    X = _search_block(prob, 20, seed=11)
    Q, _, _ = oqr.cholqr2(X)
    A, B = dev_blocks(prob)
    s1 = PHSolver(A, B, prob.nev, prob.nex, rr_max_sweeps=1)
    with pytest.raises(ChasePHError) as e:
        s1.oblique_rr(to_dev(Q))
    assert e.value.status == _lib.ERR_EIG
    s1.close()
    s40 = PHSolver(A, B, prob.nev, prob.nex)
    ritz, _, _ = s40.oblique_rr(to_dev(Q))
    lam_ref, _, _ = rayleigh_ritz.oblique_rr(prob.A, prob.B, Q)
    assert np.allclose(ritz, lam_ref, rtol=1e-11, atol=0)
    s40.close()


@pytest.mark.parametrize("kh", [6, 32])
@pytest.mark.parametrize("eps", [1e-2, 1e-3, 1e-5, 1e-8, 1e-13])
def test_rr_near_diagonal_quotient(prob, solver80, kh, eps):
    # a search block eps away from an invariant subspace: the quotient starts
    # nearly diagonal, so GEMM refinement steps take the place of some or all
    # of the Jacobi sweeps.  Same bounds as for a random block.
    print_case("rr_near_diagonal", m=prob.m, k=2 * kh, eps=eps)
    lam, Vp = dense.dense_ph_eig(prob.A, prob.B)
    X = np.concatenate([Vp[:, :kh], ham.apply_k_conj(Vp[:, :kh])], axis=1)
    X = X / np.linalg.norm(X, axis=0)
    X = X + eps * complex_normal(np.random.default_rng(kh), X.shape) / np.sqrt(prob.n)
    Q, _, _ = oqr.cholqr2(X)
    lam_ref, _, _ = rayleigh_ritz.oblique_rr(prob.A, prob.B, Q)
    ritz, Z, T = solver80.oblique_rr(to_dev(Q))
    assert np.allclose(ritz, lam_ref, rtol=1e-11, atol=0)
    Vh = to_host(solver80.residuals(to_dev(Q), T, Z, ritz)[0])
    R = ham.apply_h(prob.A, prob.B, Vh) - Vh * ritz[None, :]
    assert np.max(np.abs(Q.conj().T @ ham.apply_s(R))) < 1e-11
    G = Vh.conj().T @ ham.apply_s(ham.apply_h(prob.A, prob.B, Vh))  # V^H S H V is diagonal
    d = np.sqrt(np.abs(np.diag(G)))
    assert np.max(np.abs(G / np.outer(d, d) - np.eye(kh))) < 1e-11


# the same further from diagonal, around the limits of the refinement steps
# (||o_ij / (g_jj - g_ii)||_F of 0.035 and 0.095): the series to E^8, to E^12, sweeps
@pytest.mark.parametrize("kh", [6, 32])
@pytest.mark.parametrize("eps", [3e-2, 6e-2, 0.1, 0.2, 0.4])
def test_rr_refinement_limits(prob, solver80, kh, eps):
    test_rr_near_diagonal_quotient(prob, solver80, kh, eps)


def _unit_ritz(Q, Z):
    V = Q @ Z
    return V / np.linalg.norm(V, axis=0)[None, :]


@pytest.fixture(scope="module")
def solver260(prob):
    """Handle with nevex = 130: Rayleigh-Ritz blocks of up to 260 columns."""
    A, B = dev_blocks(prob)
    s = PHSolver(A, B, 100, 30)
    yield s
    s.close()


@pytest.mark.parametrize("kh", [1, 2, 20, 40, 130])
def test_oblique_rr_backup_matches_oracle(prob, solver, solver80, solver260, kh):
    # Section 5.3 back-up quotient on a filtered search block; k = 2 .. 260
    # (Hessenberg reduction over ragged 64-row groups, QR iteration, back-
    # substitution over up to five 64-thread groups)
    s = solver if kh <= 20 else (solver80 if kh <= 40 else solver260)
    print_case("oblique_rr_backup", m=prob.m, k=2 * kh)
    X = _search_block(prob, kh, seed=6)
    Q, _, _ = oqr.cholqr2(X)
    lam_ref, Z_ref, T_ref = rayleigh_ritz.oblique_rr_backup(prob.A, prob.B, Q)
    Qd = to_dev(Q)
    ritz, Z, T = s.oblique_rr_backup(Qd)
    assert np.allclose(ritz, lam_ref, rtol=1e-10, atol=0)
    assert np.max(np.abs(to_host(T) - T_ref)) < 1e-12 * np.max(np.abs(T_ref))
    Vref = _unit_ritz(Q, Z_ref)
    V = align_columns(_unit_ritz(Q, to_host(Z)), Vref)
    assert np.max(np.abs(V - Vref)) < 1e-8
    Vr, res = s.residuals(Qd, T, Z, ritz)
    rref = ores.residual_norms(prob.A, prob.B, ores.back_transform(Q, Z_ref), lam_ref)
    assert np.allclose(res, rref, rtol=1e-6, atol=1e-12)


def test_oblique_rr_backup_exact_invariant_subspace(prob, solver):
    lam, Vp = dense.dense_ph_eig(prob.A, prob.B)
    X = np.concatenate([Vp[:, :6], ham.apply_k_conj(Vp[:, :6])], axis=1)
    Q, _, _ = oqr.cholqr2(X)
    ritz, Z, T = solver.oblique_rr_backup(to_dev(Q))
    assert np.allclose(ritz, lam[:6], rtol=1e-11)


def test_oblique_rr_backup_recovers_exact_pair_when_qsq_singular():
    # Q^H S Q with a 2 x 2 zero block: Alg. 2 reports the singularity, the
    # back-up quotient returns the exact pair in range(Q)
    A, B, Q, lam_exact = decoupled_singular_case()
    print_case("oblique_rr_backup_singular", m=A.shape[0], k=4)
    p = make_problem(A.shape[0], lambda rng, mm: rng.uniform(1.0, 2.0, mm), 0.1, 1, 1, 4, 1e-8)
    p.A, p.B = A, B
    Ad, Bd = dev_blocks(p)
    s = PHSolver(Ad, Bd, 1, 1)
    with pytest.raises(ChasePHError) as e:
        s.oblique_rr(to_dev(Q))
    assert e.value.status == _lib.ERR_SINGULAR_QSQ
    lam_ref, Z_ref, _ = rayleigh_ritz.oblique_rr_backup(A, B, Q)
    ritz, Z, T = s.oblique_rr_backup(to_dev(Q))
    assert np.allclose(ritz, lam_ref, rtol=1e-12)
    assert np.min(np.abs(ritz - lam_exact)) < 1e-12 * lam_exact


def test_oblique_rr_backup_on_s_neutral_basis(prob, solver):
    # Q^H S Q = 0: every diagonal entry is replaced by 1
    m, k = prob.m, 4
    Q = np.zeros((prob.n, k), dtype=np.complex128)
    for j in range(k):
        Q[j, j] = Q[m + j, j] = 1 / np.sqrt(2)
    lam_ref, _, _ = rayleigh_ritz.oblique_rr_backup(prob.A, prob.B, Q)
    ritz, _, _ = solver.oblique_rr_backup(to_dev(Q))
    assert np.allclose(ritz, lam_ref, rtol=1e-12)


def test_backward_matches_oracle(prob, solver):
    from oracle import adjoint
    lam, V = dense.smallest_positive(prob.A, prob.B, 7)
    g = np.random.default_rng(2).standard_normal(7)
    GA_ref, GB_ref = adjoint.eigval_grad(V, g)
    GA, GB = solver.eigval_backward(to_dev(V), g)
    GA, GB = to_host(GA), to_host(GB)
    assert np.max(np.abs(GA - GA_ref)) < 1e-12 * np.max(np.abs(GA_ref))
    assert np.max(np.abs(GB - GB_ref)) < 1e-12 * np.max(np.abs(GB_ref))


# ------------------------------------------------------------ error paths
def test_argument_errors(solver, prob):
    X = to_dev(np.zeros((prob.n, 3)))
    with pytest.raises(ChasePHError) as e:
        solver.oblique_rr(X)          # odd k
    assert e.value.status == _lib.ERR_ARG
    W = to_dev(np.ones((prob.n, 3)))
    with pytest.raises(ChasePHError) as e:
        solver.filter(W, 1.0, 2.0, 5.0, degs=[3, 2, 4])   # not sorted
    assert e.value.status == _lib.ERR_ARG
    with pytest.raises(ChasePHError) as e:
        solver.filter(W, 2.0, 1.0, 5.0)                   # mu order
    assert e.value.status == _lib.ERR_ARG


def test_not_definite_detected():
    # SH indefinite: ||B||_2 = 2 min d.  A block containing an eigenvector of
    # SH with a negative eigenvalue makes Q^H S H Q indefinite.
    p = make_problem(64, lambda rng, mm: rng.uniform(1.0, 2.0, mm), 2.0, 2, 2, 4, 1e-8)
    SH = ham.assemble_sh(p.A, p.B)
    w, U = np.linalg.eigh(SH)
    assert w[0] < 0
    X = np.concatenate([U[:, :1], ham.apply_k_conj(U[:, :1])], axis=1)
    Q, _, _ = oqr.cholqr2(X)
    A, B = dev_blocks(p)
    s = PHSolver(A, B, 2, 2)
    with pytest.raises(ChasePHError) as e:
        s.oblique_rr(to_dev(Q))
    assert e.value.status == _lib.ERR_NOT_DEFINITE


def test_singular_qsq_detected(prob, solver):
    # S-neutral basis (Section 4.6): Q^H S Q = 0
    m, k = prob.m, 4
    Q = np.zeros((prob.n, k), dtype=np.complex128)
    for j in range(k):
        Q[j, j] = Q[m + j, j] = 1 / np.sqrt(2)
    with pytest.raises(ChasePHError) as e:
        solver.oblique_rr(to_dev(Q))
    assert e.value.status == _lib.ERR_SINGULAR_QSQ


# c128 products in real coordinates: rows around the 32- and 128-row groups,
# odd m (a quad of reals half empty), columns around the 16-column fragments,
# degrees that end in either buffer, a leading dimension above n.  Every value
# is a sum of at most 2n products and the degrees are small: 1e-11 of the
# column norm as for the other c128 filters
@pytest.mark.parametrize("m,k", [(1, 1), (3, 2), (17, 8), (33, 9), (63, 24), (64, 25), (65, 40), (129, 65), (321, 130)])
def test_filter_fp64_edges(m, k):
    print_case("filter_fp64_edges", m=m, k=k)
    p = problem(m=m, seed=m, nev=1, nex=0)
    A, B = dev_blocks(p)
    s = PHSolver(A, B, k, 0)
    rng = np.random.default_rng(m + k)
    W = complex_normal(rng, (p.n, k))
    degs = sorted([1, 2, 3, 4, 5][j % 5] for j in range(k))
    buf = empty_cm(p.n + 3, k)
    Wd = buf[: p.n]
    Wd.copy_(to_dev(W))
    s.filter(Wd, 1.0, 2.5, 6.0, degs=degs, prec=FP64)
    ref = chebyshev.chebyshev_filter(p.A, p.B, W, np.array(degs), 1.0, 2.5, 6.0)
    err = np.linalg.norm(to_host(Wd) - ref, axis=0) / np.linalg.norm(ref, axis=0)
    assert np.max(err) < 1e-11, err
    a = complex_normal(rng, (m, k))
    X = np.concatenate([a, a.conj()], axis=0)
    Y = to_host(s.apply_h(to_dev(X), prec=_lib.FP64_KREAL))
    ref = ham.apply_h(p.A, p.B, X)
    assert np.max(np.abs(Y - ref)) <= 1e-12 * np.max(np.abs(ref))


# every tile width (at most 8, 4, 2, 1 column fragments) and parts that end
# inside a strip, through the epilogue of the recurrence
@pytest.mark.parametrize("plan", ["0,1", "0,3", "0,7", "1,2", "1,5", "2,3", "3,1", "3,4"])
def test_filter_fp64_every_tile_plan(prob, plan, monkeypatch):
    k = 77
    print_case("filter_fp64_plan", m=prob.m, k=k, plan=plan)
    monkeypatch.setenv("CHASE_PH_APPLY_PLAN", plan)
    A, B = dev_blocks(prob)
    s = PHSolver(A, B, k, 0)
    mu1, mu_nevex, mu_n = _mus(prob)
    rng = np.random.default_rng(77)
    W = complex_normal(rng, (prob.n, k))
    degs = [2] * 30 + [3] * 30 + [5] * 17
    Wd = to_dev(W)
    s.filter(Wd, mu1, mu_nevex, mu_n, degs=degs, prec=FP64)
    ref = chebyshev.chebyshev_filter(prob.A, prob.B, W, np.array(degs), mu1, mu_nevex, mu_n)
    err = np.linalg.norm(to_host(Wd) - ref, axis=0) / np.linalg.norm(ref, axis=0)
    assert np.max(err) < 1e-11, err


# every shape of the short products, at sizes with fewer K slabs of 8 than a
# workgroup has waves (m = 5), a last strip and a last column tile that are cut
# off (m = 13, 75) and full ones (m = 64, 2 k = 64), general and K-real
# columns, through the plain and the recurrence's epilogue
@pytest.mark.parametrize("plan", ["4,1", "5,1", "6,1", "7,1", "8,1", "9,1"])
@pytest.mark.parametrize("m,k", [(5, 2), (13, 9), (64, 32), (75, 41), (75, 57)])
def test_short_products_every_shape(m, k, plan, monkeypatch):
    print_case("short_products", m=m, k=k, plan=plan)
    monkeypatch.setenv("CHASE_PH_APPLY_PLAN", plan)
    p = problem(m=m, seed=m, nev=1, nex=0)
    A, B = dev_blocks(p)
    s = PHSolver(A, B, k, 0)
    rng = np.random.default_rng(m + k)
    X = complex_normal(rng, (p.n, k))
    ref = ham.apply_h(p.A, p.B, X)
    assert np.max(np.abs(to_host(s.apply_h(to_dev(X))) - ref)) <= 1e-12 * np.max(np.abs(ref))
    a = complex_normal(rng, (m, k))
    X = np.concatenate([a, a.conj()], axis=0)
    ref = ham.apply_h(p.A, p.B, X)
    Y = to_host(s.apply_h(to_dev(X), prec=_lib.FP64_KREAL))
    assert np.max(np.abs(Y - ref)) <= 1e-12 * np.max(np.abs(ref))
    mu1, mu_nevex, mu_n = 0.9, 2.0, 1.2 * np.max(np.linalg.eigvalsh(ham.assemble_sh(p.A, p.B)))
    W = complex_normal(rng, (p.n, k))
    degs = [2] * (k // 2) + [5] * (k - k // 2)
    Wd = to_dev(W)
    s.filter(Wd, mu1, mu_nevex, mu_n, degs=degs, prec=FP64)
    ref = chebyshev.chebyshev_filter(p.A, p.B, W, np.array(degs), mu1, mu_nevex, mu_n)
    err = np.linalg.norm(to_host(Wd) - ref, axis=0) / np.linalg.norm(ref, axis=0)
    assert np.max(err) < 1e-11, err
    s.close()


# c128 GEMMs of the QR and Rayleigh-Ritz steps: sizes around the 32-row waves,
# the 64-row tiles and the 8-row K slabs, with odd m (K and the sign flip of S
# end inside a slab), against the oracle at the tolerances of the larger cases
@pytest.mark.parametrize("m,k", [(19, 2), (33, 16), (67, 32), (130, 34), (261, 66), (389, 130)])
def test_qr_rr_residuals_gemm_edges(m, k):
    print_case("gemm_edges", m=m, k=k)
    p = problem(m=m, seed=m, nev=1, nex=0)
    A, B = dev_blocks(p)
    s = PHSolver(A, B, k // 2, 0)
    rng = np.random.default_rng(m)
    W = complex_normal(rng, (p.n, k // 2))
    W[m:] *= 1e-3
    X = np.concatenate([W, ham.apply_k_conj(W)], axis=1)
    Qd = to_dev(X)
    Rd, _ = s.qr(Qd)
    Q, R = to_host(Qd), to_host(Rd)
    Qr, Rr = np.linalg.qr(X)
    ph = np.diag(Rr) / np.abs(np.diag(Rr))
    assert np.max(np.abs(Q - Qr * ph)) < 1e-9
    assert np.max(np.abs(R - Rr * ph.conj()[:, None])) < 1e-9 * np.max(np.abs(Rr))
    ritz, Z, T = s.oblique_rr(Qd)
    ref_ritz = rayleigh_ritz.oblique_rr(p.A, p.B, Q)[0]
    assert np.max(np.abs(ritz - ref_ritz) / np.abs(ref_ritz)) < 1e-11
    V, res = s.residuals(Qd, T, Z, ritz)
    V = to_host(V)
    assert np.max(np.abs(np.linalg.norm(V, axis=0) - 1)) < 1e-12
    hv = ham.apply_h(p.A, p.B, V) - V * ritz[None, :]
    assert np.max(np.abs(np.linalg.norm(hv, axis=0) - res)) < 1e-11


# Cholesky factor and inverse of the blocked kernel through the QR of 64-column
# blocks: sizes at, below and above one and two blocks, where R = L^H and
# Q = X L^{-H}; the unique QR at 1e-11 of its scale (cond(X) below 100)
@pytest.mark.parametrize("k", [2, 62, 64, 66, 126, 128, 130, 192])
def test_qr_block_edges(k):
    print_case("qr_block_edges", k=k)
    p = problem(m=200, seed=3, nev=1, nex=0)
    A, B = dev_blocks(p)
    s = PHSolver(A, B, (k + 1) // 2, 0)
    rng = np.random.default_rng(k)
    X = complex_normal(rng, (p.n, k)) * np.linspace(0.1, 1.0, k)[None, :]
    Qd = to_dev(X)
    Rd, variant = s.qr(Qd)
    assert variant == 0
    Q, R = to_host(Qd), to_host(Rd)
    Qr, Rr = np.linalg.qr(X)
    ph = np.diag(Rr) / np.abs(np.diag(Rr))
    assert np.max(np.abs(Q - Qr * ph)) < 1e-11
    assert np.max(np.abs(R - Rr * ph.conj()[:, None])) < 1e-11 * np.max(np.abs(Rr))
    assert np.max(np.abs(np.tril(R, -1))) == 0.0


# k x k x k products around the sizes where the small-product kernel changes
# its tile (386: 16 x 16 outputs, 434 and 450: 32 x 32) and gives way to the
# large one (514), all with cut-off tiles and K slabs; bounds as above
@pytest.mark.parametrize("k", [386, 434, 450, 514])
def test_qr_product_shapes(k):
    print_case("qr_product_shapes", k=k)
    p = problem(m=600, seed=4, nev=1, nex=0)
    A, B = dev_blocks(p)
    s = PHSolver(A, B, (k + 1) // 2, 0)
    rng = np.random.default_rng(k)
    X = complex_normal(rng, (p.n, k)) * np.linspace(0.1, 1.0, k)[None, :]
    Qd = to_dev(X)
    Rd, variant = s.qr(Qd)
    assert variant == 0
    Q, R = to_host(Qd), to_host(Rd)
    Qr, Rr = np.linalg.qr(X)
    ph = np.diag(Rr) / np.abs(np.diag(Rr))
    assert np.max(np.abs(Q - Qr * ph)) < 1e-11
    assert np.max(np.abs(R - Rr * ph.conj()[:, None])) < 1e-11 * np.max(np.abs(Rr))
    assert np.max(np.abs(np.tril(R, -1))) == 0.0
    s.close()


# c128 products where the workspace decides the cut: sizes that ran on whole
# strips for want of room (m = 1050, 2 k = 544, 1450 with 576), a forced split whose
# partial sums do not fit (m = 850: "0,64" wants 14 strips in 64 parts of 8
# column tiles, whole strips), one whose do in part (4 tiles), and exactly one
# workgroup of the widest tiles per CU (m = 2000, 2 k = 1024).  Each against H X
# formed by matmul, a sum of 2n products: 1e-12 of the largest entry
@pytest.mark.parametrize("m,k,plan", [(1050, 272, None), (1450, 288, None), (850, 512, "0,64"), (850, 256, "0,64"),
                                      (2000, 512, None)])
def test_apply_h_fp64_workspace(m, k, plan, monkeypatch):
    print_case("apply_h_fp64_workspace", m=m, k=k, plan=plan)
    if plan:
        monkeypatch.setenv("CHASE_PH_APPLY_PLAN", plan)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(m + k)

    def normal(*shape):
        return torch.complex(torch.randn(shape, dtype=torch.float64, device="cuda", generator=gen),
                             torch.randn(shape, dtype=torch.float64, device="cuda", generator=gen))

    A, B = normal(m, m), normal(m, m)
    A, B = (A + A.mH).contiguous(), (B + B.T).contiguous()
    x, y = normal(m, k), normal(m, k)
    ref = torch.cat([A @ x + B @ y, -(B.conj() @ x) - A.conj() @ y])
    s = PHSolver(A, B, 8, 8)
    Y = s.apply_h(torch.cat([x, y]).T.contiguous().T)
    assert (Y - ref).abs().max() <= 1e-12 * ref.abs().max()
    s.close()


# c128 products of more columns than one launch takes (2 x 12000 reals: 1280):
# 1300 real columns of a product and of the recurrence, whose even and odd
# degrees end in different buffers.  Against matmul at the bounds of the
# smaller cases
def test_c128_products_in_column_groups():
    m, k = 12000, 650
    print_case("column_groups", m=m, k=k)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7)

    def normal(*shape):
        return torch.complex(torch.randn(shape, dtype=torch.float64, device="cuda", generator=gen),
                             torch.randn(shape, dtype=torch.float64, device="cuda", generator=gen))

    A = torch.diag(torch.linspace(1.0, 5.0, m, dtype=torch.float64, device="cuda")).to(torch.complex128)
    B = normal(m, m) * (0.1 / m ** 0.5)
    B = (B + B.T).contiguous()
    X = normal(2 * m, k)

    def hx(x):
        u, v = x[:m], x[m:]
        return torch.cat([A @ u + B @ v, -(B.conj() @ u) - A.conj() @ v])

    s = PHSolver(A, B, k, 0)
    ref = hx(X)
    assert (s.apply_h(X.T.contiguous().T) - ref).abs().max() <= 1e-12 * ref.abs().max()
    mu1, mu_nevex, mu_n = 0.8, 2.0, 6.0
    c, e = 0.5 * (mu_n ** 2 + mu_nevex ** 2), 0.5 * (mu_n ** 2 - mu_nevex ** 2)
    s1 = e / (mu1 ** 2 - c)
    W1 = (s1 / e) * (hx(ref) - c * X)
    s2 = 1.0 / (2.0 / s1 - s1)
    W2 = (2.0 * s2 / e) * (hx(hx(W1)) - c * W1) - s1 * s2 * X
    ref = torch.cat([W1[:, :30], W2[:, 30:]], dim=1)
    W = X.T.contiguous().T
    s.filter(W, mu1, mu_nevex, mu_n, degs=[1] * 30 + [2] * (k - 30), prec=FP64)
    err = torch.linalg.vector_norm(W - ref, dim=0) / torch.linalg.vector_norm(ref, dim=0)
    assert err.max() < 1e-11, err.max()
    s.close()


# a quotient large enough (k = 3072) that the Jacobi rounds are applied in place,
# their rotations found in launches of their own: Galerkin condition, diagonal
# V^H S H V and residuals, formed by matmul; sums of 3200 products, the bounds of
# the small quotients
def test_rr_rounds_in_place():
    m, kh = 1600, 1536
    print_case("rr_in_place", m=m, k=2 * kh)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(11)

    def normal(*shape):
        return torch.complex(torch.randn(shape, dtype=torch.float64, device="cuda", generator=gen),
                             torch.randn(shape, dtype=torch.float64, device="cuda", generator=gen))

    E = normal(m, m) * (0.2 / m ** 0.5)
    A = (torch.diag(torch.linspace(1.0, 5.0, m, dtype=torch.float64, device="cuda")).to(torch.complex128) + E + E.mH)
    B = normal(m, m) * (0.05 / m ** 0.5)
    A, B = A.contiguous(), (B + B.T).contiguous()
    W = normal(2 * m, kh)
    W[m:] *= 1e-3
    X = torch.cat([W, torch.cat([W[m:].conj(), W[:m].conj()])], dim=1).T.contiguous().T
    s = PHSolver(A, B, kh, 0)
    s.qr(X)
    ritz, Z, T = s.oblique_rr(X)
    lam = torch.from_numpy(np.asarray(ritz)).cuda()
    assert bool((lam[1:] >= lam[:-1]).all()) and lam[0] > 0
    HX = torch.cat([A @ X[:m] + B @ X[m:], -(B.conj() @ X[:m]) - A.conj() @ X[m:]])
    assert (T - HX).abs().max() <= 1e-12 * HX.abs().max()
    V = X @ Z
    nu = torch.linalg.vector_norm(V, dim=0)
    V, HV = V / nu, (HX @ Z) / nu
    R = HV - V * lam[None, :]
    R[m:] *= -1.0
    assert (X.mH @ R).abs().max() < 1e-11
    HV[m:] *= -1.0
    G = V.mH @ HV
    d = torch.diagonal(G).real.abs().sqrt()
    G = G / torch.outer(d, d) - torch.eye(kh, dtype=G.dtype, device="cuda")
    assert G.abs().max() < 1e-11
    s.close()


# A search block eps away from an invariant subspace and the number of sweeps that
# a cyclic Jacobi method needs from its quotient (counted in numpy): enough as the
# limit, also where refinement steps, which need one more than sweeps do from
# ||o_ij / (g_jj - g_ii)||_F of 0.1 on, take the place of the last ones
@pytest.mark.parametrize("kh,eps,limit", [(6, 1e-3, 3), (20, 1e-2, 3), (32, 1e-2, 3), (32, 3e-2, 4), (32, 0.1, 5)])
def test_rr_sweep_limit_of_a_cyclic_jacobi(prob, kh, eps, limit):
    print_case("rr_sweep_limit", m=prob.m, k=2 * kh, eps=eps, limit=limit)
    lam, Vp = dense.dense_ph_eig(prob.A, prob.B)
    X = np.concatenate([Vp[:, :kh], ham.apply_k_conj(Vp[:, :kh])], axis=1)
    X = X / np.linalg.norm(X, axis=0)
    X = X + eps * complex_normal(np.random.default_rng(kh), X.shape) / np.sqrt(prob.n)
    Q, _, _ = oqr.cholqr2(X)
    A, B = dev_blocks(prob)
    s = PHSolver(A, B, 32, 0, rr_max_sweeps=limit)
    ritz, _, _ = s.oblique_rr(to_dev(Q))
    assert np.allclose(ritz, rayleigh_ritz.oblique_rr(prob.A, prob.B, Q)[0], rtol=1e-11, atol=0)
    s.close()


def test_singular_qsq_leaves_the_outputs_alone(prob, solver):
    # the refused call writes neither the Ritz values nor Z
    import ctypes
    print_case("singular_qsq_outputs", m=prob.m, k=4)
    m, k = prob.m, 4
    Q = np.zeros((prob.n, k), dtype=np.complex128)
    for j in range(k):
        Q[j, j] = Q[m + j, j] = 1 / np.sqrt(2)
    Q = to_dev(Q)
    Z, T = torch.full((k // 2, k), 7.0 - 3.0j, dtype=torch.complex128, device="cuda").T, empty_cm(prob.n, k)
    ritz = (ctypes.c_double * (k // 2))(5.0, 6.0)
    st = _lib.load().chase_ph_oblique_rr(solver._h, k, Q.data_ptr(), prob.n, ritz, Z.data_ptr(), k, T.data_ptr(), prob.n)
    assert st == _lib.ERR_SINGULAR_QSQ
    assert list(ritz) == [5.0, 6.0]
    assert bool((Z == 7.0 - 3.0j).all())


# the recurrence keeps the product of each degree in the buffer that other
# products pack into: whatever those left there (NaN of more columns, so at other
# places), also past row 2m, the filter's columns do not see it
@pytest.mark.parametrize("m,k", [(5, 3), (33, 9), (64, 7), (75, 20)])
def test_filter_fp64_after_a_product_of_nan(m, k):
    print_case("filter_after_nan", m=m, k=k)
    p = problem(m=m, seed=m, nev=1, nex=0)
    A, B = dev_blocks(p)
    s = PHSolver(A, B, k, 0)
    s.apply_h(torch.full((512, p.n), float("nan"), dtype=torch.complex128, device="cuda").T)
    rng = np.random.default_rng(m)
    W = complex_normal(rng, (p.n, k))
    degs = [1 + j % 3 for j in range(k)]
    degs.sort()
    Wd = to_dev(W)
    s.filter(Wd, 1.0, 2.5, 6.0, degs=degs, prec=FP64)
    ref = chebyshev.chebyshev_filter(p.A, p.B, W, np.array(degs), 1.0, 2.5, 6.0)
    err = np.linalg.norm(to_host(Wd) - ref, axis=0) / np.linalg.norm(ref, axis=0)
    assert np.max(err) < 1e-11, err
    s.close()


# both kinds of stores of the adjoint: columns that start on 64 bytes of outputs of up
# to 32 MiB (m = 64, 1024) or of many eigenpairs (160), and all others, by m, by the
# leading dimension and by the first element; pads and neighbours stay as they were.  Sums of nev products of
# unit vectors' entries: 1e-12 of the largest entry
@pytest.mark.parametrize("m,nev,pad,shift", [(64, 5, 0, 0), (64, 5, 1, 0), (64, 5, 4, 1), (65, 4, 0, 0), (130, 7, 2, 4),
                                             (1024, 3, 0, 0), (1028, 3, 0, 0), (1028, 161, 0, 0)])
def test_backward_stores(m, nev, pad, shift):
    import ctypes
    print_case("backward_stores", m=m, nev=nev, pad=pad, shift=shift)
    rng = np.random.default_rng(m + nev)
    V = complex_normal(rng, (2 * m, nev))
    V[m:] *= 0.3
    V /= np.linalg.norm(V, axis=0)
    g = rng.standard_normal(nev)
    x, y = V[:m], V[m:]
    gt = g / (np.sum(np.abs(x) ** 2, axis=0) - np.sum(np.abs(y) ** 2, axis=0))
    refA = (x * gt) @ x.conj().T + (y.conj() * gt) @ y.T
    refB = (x * gt) @ y.conj().T + (y.conj() * gt) @ x.T
    ldg = m + pad
    A, B = (torch.full((ldg * m + shift,), 9.0 + 1.0j, dtype=torch.complex128, device="cuda") for _ in range(2))
    Vd = to_dev(V)
    hg = (ctypes.c_double * nev)(*g)
    st = _lib.load().chase_ph_eigval_backward_noalloc(m, nev, Vd.data_ptr(), 2 * m, hg, A.data_ptr() + 16 * shift,
                                                      B.data_ptr() + 16 * shift, ldg,
                                                      torch.cuda.current_stream().cuda_stream)
    assert st == _lib.OK
    for out, ref in ((A, refA), (B, refB)):
        assert bool((out[:shift] == 9.0 + 1.0j).all())
        cols = out[shift:].reshape(m, ldg).cpu().numpy()  # a row: one column
        assert np.all(cols[:, m:] == 9.0 + 1.0j)
        assert np.max(np.abs(cols[:, :m].T - ref)) <= 1e-12 * np.max(np.abs(ref))
