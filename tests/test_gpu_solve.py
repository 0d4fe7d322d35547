"""End-to-end parity of chase_ph_solve (Alg. 3) and of the autograd path
against the CPU oracle.  Bar (spec tolerances): eigenvalues within
1e-10 relative of the dense oracle on the FP64 path and 1e-9 on the mixed
path; every returned pair has residual <= tol."""
import os

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from oracle import adjoint, dense, hamiltonian as ham, residuals as ores, inertia
from paper_2601_10557_amd import FP64, MIXED, ChasePHError, PHSolver, eigsh_ph
from paper_2601_10557_amd import _lib
from synth import config_problem, make_problem
from gpu_helpers import dev_blocks, print_case, to_dev, to_host

GOLDEN = os.path.join(os.path.dirname(__file__), "golden")


def _check_solution(p, ev, V, res, ref, rtol):
    assert len(ev) == p.nev
    assert np.all(np.diff(ev) > 0)
    rel = np.abs(ev - ref[: p.nev]) / ref[: p.nev]
    assert np.max(rel) <= rtol, np.max(rel)
    Vh = to_host(V)
    r = ores.residual_norms(p.A, p.B, Vh, ev)
    assert np.all(r <= p.tol * 1.5), np.max(r)
    assert np.all(res <= p.tol)
    D = Vh.conj().T @ ham.apply_s(Vh)                     # eq. 3.5: V^H S V diagonal
    off = D - np.diag(np.diag(D))
    assert np.max(np.abs(off)) < 1e-7
    assert np.all(np.real(np.diag(D)) > 0)


@pytest.fixture(scope="module")
def cfg0():
    p = config_problem(0)
    lam, _ = dense.dense_ph_eig(p.A, p.B)
    return p, lam


def _solve(p, **kw):
    A, B = dev_blocks(p)
    s = PHSolver(A, B, p.nev, p.nex, deg=p.deg, tol=kw.pop("tol", p.tol), **kw)
    return s, s.solve(to_dev(p.w0_raw), to_dev(p.lanczos_raw))


def test_lanczos_estimates_match_oracle(cfg0):
    # Section 4.1 spectral estimates of the solver (26 steps x 4 runs on the
    # gamma-scaled starts) against the oracle's on the same starts; rounding
    # perturbations of the starts move them by ~1e-13 relative
    from oracle import lanczos, solver as osolver
    p, _ = cfg0
    print_case("lanczos_estimates", cfg=0, m=p.m)
    A, B = dev_blocks(p)
    s = PHSolver(A, B, p.nev, p.nex, deg=p.deg, tol=p.tol, max_iter=1)
    _, _, _, info = s.solve(to_dev(p.w0_raw), to_dev(p.lanczos_raw), raise_on_noconv=False)
    s.close()
    ref = lanczos.spectral_estimates(p.A, p.B, osolver.init_block(p.lanczos_raw, 1e-3), 26, p.nev + p.nex)
    assert np.allclose([info.mu1, info.mu_nevex0, info.mu_n], ref, rtol=1e-9, atol=0)


def test_solve_fp64_config0(cfg0):
    p, lam = cfg0
    print_case("solve_fp64", cfg=0, m=p.m)
    _, (ev, V, res, info) = _solve(p, precision=FP64)
    _check_solution(p, ev, V, res, lam, 1e-10)
    assert info.iterations <= 25


def test_solve_mixed_config0(cfg0):
    p, lam = cfg0
    print_case("solve_mixed", cfg=0, m=p.m)
    p.tol = 1e-9
    try:
        _, (ev, V, res, info) = _solve(p, precision=MIXED)
        _check_solution(p, ev, V, res, lam, 1e-9)
        assert info.filter_flops_fp32 > 0
    finally:
        p.tol = 1e-10


def test_solve_per_vector_degrees(cfg0):
    p, lam = cfg0
    print_case("solve_optdeg", cfg=0, m=p.m)
    _, (ev, V, res, info) = _solve(p, precision=FP64, opt_deg=True, deg_min=8, deg_max=20)
    _check_solution(p, ev, V, res, lam, 1e-10)


@pytest.mark.parametrize("prec", [FP64, MIXED])
def test_solve_backup_rr_every_iteration(cfg0, prec):
    # the non-hermitian back-up quotient of Section 5.3 in every iteration
    p, lam = cfg0
    print_case("solve_backup_rr", cfg=0, m=p.m, prec=prec)
    tol0 = p.tol
    p.tol = 1e-10 if prec == FP64 else 1e-9
    try:
        _, (ev, V, res, info) = _solve(p, precision=prec, rr_backup=True, max_iter=40)
        _check_solution(p, ev, V, res, lam, p.tol)
        assert info.backup_rr_used == info.iterations
    finally:
        p.tol = tol0


def test_solve_zero_start_column_takes_householder_qr(cfg0):
    # a zero column in the start block stays zero through the filter, so the
    # first search block is rank deficient: QR falls back to Householder and
    # the solve still reaches the dense oracle's eigenvalues
    p, lam = cfg0
    print_case("solve_householder", cfg=0, m=p.m)
    w0 = np.array(p.w0_raw, copy=True)
    w0[:, 5] = 0
    A, B = dev_blocks(p)
    s = PHSolver(A, B, p.nev, p.nex, deg=p.deg, tol=p.tol, precision=FP64)
    ev, V, res, info = s.solve(to_dev(w0), to_dev(p.lanczos_raw))
    assert info.householder_qr_used >= 1
    _check_solution(p, ev, V, res, lam, 1e-10)


def test_solve_b_zero_is_tda():
    # Section 1.1: B = 0 reduces to A X = X Omega
    p = make_problem(200, lambda rng, m: rng.uniform(1.0, 5.0, m), 0.3, 8, 6, 12, 1e-10, seed=3)
    p.B = np.zeros_like(p.B)
    print_case("solve_b0", m=p.m)
    _, (ev, V, res, info) = _solve(p)
    assert np.allclose(ev, np.sort(p.d)[:8], rtol=1e-10)
    assert np.max(np.abs(to_host(V)[200:])) < 1e-8


@pytest.mark.parametrize("m,nev,nex,prec", [(301, 1, 3, FP64), (257, 5, 3, MIXED), (130, 12, 4, FP64)])
def test_solve_small_and_odd_shapes(m, nev, nex, prec):
    # odd m (no direct-to-LDS tiles), a single wanted pair, m not a multiple
    # of any tile: the solver still reaches the dense eigenvalues (the CPU
    # oracle converges on the same draws in 32, 33 and 8 iterations)
    p = make_problem(m, lambda rng, mm: rng.uniform(1.0, 5.0, mm), 0.3, nev, nex, 12, 1e-10, seed=7)
    print_case("solve_shape", m=m, nev=nev, nex=nex, prec=prec)
    lam, _ = dense.dense_ph_eig(p.A, p.B)
    tol = 1e-10 if prec == FP64 else 1e-9
    p.tol = tol
    _, (ev, V, res, info) = _solve(p, precision=prec, max_iter=40)
    _check_solution(p, ev, V, res, lam, tol)


def test_solve_no_convergence_partial(cfg0):
    p, lam = cfg0
    A, B = dev_blocks(p)
    s = PHSolver(A, B, p.nev, p.nex, deg=4, tol=1e-13, max_iter=1)
    with pytest.raises(ChasePHError) as e:
        s.solve(to_dev(p.w0_raw), to_dev(p.lanczos_raw))
    assert e.value.status == _lib.ERR_NO_CONVERGENCE
    ev, V, res, info = s.solve(to_dev(p.w0_raw), to_dev(p.lanczos_raw), raise_on_noconv=False)
    assert info.iterations == 1 and len(ev) == info.locked


def test_solve_config1_fp64_and_mixed():
    """Full-size m=4000 workload: both precisions, and the mixed path with the
    back-up quotient of Section 5.3 in every iteration (k up to 520), against
    the stored dense oracle eigenvalues (tests/golden, written by
    make_dense_reference.py)."""
    path = os.path.join(GOLDEN, "dense_evals_config1_seed0.txt")
    if not os.path.exists(path):
        pytest.skip("golden file missing")
    ref = np.loadtxt(path)
    p = config_problem(1)
    print_case("solve_config1", m=p.m)
    A, B = dev_blocks(p)
    W0, Lz = to_dev(p.w0_raw), to_dev(p.lanczos_raw)
    out = {}
    for prec, backup in ((FP64, False), (MIXED, False), (MIXED, True)):
        s = PHSolver(A, B, p.nev, p.nex, deg=p.deg, tol=p.tol, precision=prec, rr_backup=backup)
        ev, V, res, info = s.solve(W0, Lz)
        rel = np.abs(ev - ref[: p.nev]) / ref[: p.nev]
        print_case("config1", prec=prec, backup=backup, iters=info.iterations, t=round(info.t_total, 3),
                   maxrel=rel.max())
        assert info.backup_rr_used == (info.iterations if backup else 0)
        assert np.max(rel) <= 1e-9
        assert np.all(res <= p.tol)
        # sampled host recomputation of residuals (8 pairs)
        idx = np.linspace(0, p.nev - 1, 8).astype(int)
        Vh = to_host(V[:, idx])
        r = ores.residual_norms(p.A, p.B, Vh, ev[idx])
        assert np.all(r <= 1.5 * p.tol)
        out[(prec, backup)] = ev
        s.close()
    assert np.max(np.abs(out[(FP64, False)] - out[(MIXED, False)]) / out[(FP64, False)]) <= 1e-9
    assert np.max(np.abs(out[(MIXED, True)] - out[(MIXED, False)]) / out[(MIXED, False)]) <= 1e-9
    # completeness by Sylvester's law of inertia (the certificate used where
    # no dense reference exists): exactly nev eigenvalues below
    # lambda_nev + delta and nev - 1 below lambda_nev - delta
    ev = out[(MIXED, False)]
    delta = 1e-3 * (ev[-1] - ev[-2])
    assert inertia.count_below(p.A, p.B, ev[-1] + delta) == p.nev
    assert inertia.count_below(p.A, p.B, ev[-1] - delta) == p.nev - 1


def test_autograd_matches_dense_adjoint_and_fd():
    p = make_problem(120, lambda rng, m: rng.uniform(1.0, 5.0, m), 0.4, 5, 5, 16, 1e-12, seed=4)
    print_case("autograd", m=p.m)
    A, B = dev_blocks(p)
    A.requires_grad_(True)
    B.requires_grad_(True)
    lam = eigsh_ph(A, B, p.nev, p.nex, to_dev(p.w0_raw), to_dev(p.lanczos_raw), deg=p.deg, tol=p.tol)
    w = torch.from_numpy(p.loss_w).cuda()
    (lam * w).sum().backward()
    GA, GB = to_host(A.grad), to_host(B.grad)
    lam_ref, Vref = dense.smallest_positive(p.A, p.B, p.nev)
    assert np.allclose(to_host(lam), lam_ref, rtol=1e-11)
    GA_ref, GB_ref = adjoint.eigval_grad(Vref, p.loss_w)
    assert np.max(np.abs(GA - GA_ref)) < 1e-8 * np.max(np.abs(GA_ref))
    assert np.max(np.abs(GB - GB_ref)) < 1e-8 * np.max(np.abs(GB_ref))
    rng = np.random.default_rng(0)
    h = 1e-6
    for _ in range(4):
        EA = rng.standard_normal((120, 120)) + 1j * rng.standard_normal((120, 120))
        EA = 0.5 * (EA + EA.conj().T)
        EB = rng.standard_normal((120, 120)) + 1j * rng.standard_normal((120, 120))
        EB = 0.5 * (EB + EB.T)
        lp, _ = dense.smallest_positive(p.A + h * EA, p.B + h * EB, p.nev)
        lm, _ = dense.smallest_positive(p.A - h * EA, p.B - h * EB, p.nev)
        fd = (p.loss_w @ lp - p.loss_w @ lm) / (2 * h)
        an = np.real(np.vdot(GA, EA)) + np.real(np.vdot(GB, EB))
        assert abs(fd - an) <= 1e-6 * max(1.0, abs(an))


@pytest.mark.parametrize("prec", [FP64, MIXED])
def test_solve_clustered_spectrum_to_convergence(prec):
    """Reduced clustered workload (80% of the eigenvalues of A in [1, 1.2],
    the rest up to 20; m = 500, nev = 10, nex = 20), per-vector degrees
    10..36, tol 1e-9, solved to convergence against the dense oracle.  The
    filter on H^2 separates the cluster from the damped interval by little
    per iteration: the oracle's own Alg. 3 takes 239 iterations here."""
    p = config_problem(2, m=500, nev=10, nex=20)
    print_case("solve_clustered", m=p.m, prec=prec)
    lam, _ = dense.dense_ph_eig(p.A, p.B)
    A, B = dev_blocks(p)
    s = PHSolver(A, B, p.nev, p.nex, deg=p.deg, tol=p.tol, precision=prec, max_iter=400, opt_deg=True,
                 deg_min=p.deg_min, deg_max=p.deg_max)
    ev, V, res, info = s.solve(to_dev(p.w0_raw), to_dev(p.lanczos_raw))
    s.close()
    print_case("solve_clustered_done", iterations=info.iterations)
    assert np.max(np.abs(ev - lam[: p.nev]) / lam[: p.nev]) <= 1e-9
    assert np.all(res <= p.tol)
    assert np.all(ores.residual_norms(p.A, p.B, to_host(V), ev) <= 1.5 * p.tol)
    assert 150 <= info.iterations <= 320
    assert 1 <= info.rr_sweeps_max < 40


def test_solve_on_wide_real_products():
    # 840 columns of 8000 reals: the orthonormalisation's Gram matrix and its
    # triangular product run on the widest tiles of the real GEMM, with cut-off
    # tiles (840 = 13 x 64 + 8).
    # Every returned pair against H V formed by matmul, and eq. 3.5
    m, nev, nex, tol = 4000, 400, 20, 1e-7
    print_case("solve_wide_real", m=m, nev=nev, nex=nex)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)

    def normal(*shape):
        return torch.complex(torch.randn(shape, dtype=torch.float64, device="cuda", generator=gen),
                             torch.randn(shape, dtype=torch.float64, device="cuda", generator=gen))

    d = torch.linspace(1.0, 9.0, m, dtype=torch.float64, device="cuda")
    B = normal(m, m) * (0.05 / m ** 0.5)
    B = (0.5 * (B + B.T)).contiguous()
    A = torch.diag(d).to(torch.complex128)
    W0 = (torch.eye(2 * m, nev + nex, dtype=torch.complex128, device="cuda") + 1e-2 * normal(2 * m, nev + nex) / m ** 0.5)
    Lz = normal(2 * m, 4)
    s = PHSolver(A, B, nev, nex, deg=20, tol=tol, max_iter=30, precision=FP64)
    ev, V, res, info = s.solve(W0.T.contiguous().T, Lz.T.contiguous().T)
    assert info.iterations > 1
    lam = torch.from_numpy(np.asarray(ev)).cuda().to(torch.complex128)
    X, Y = V[:m], V[m:]
    HV = torch.cat([A @ X + B @ Y, -(B.conj() @ X) - A.conj() @ Y])
    r = torch.linalg.vector_norm(HV - V * lam[None, :], dim=0).cpu().numpy()
    assert np.all(r <= 1.5 * tol), r.max()
    assert np.all(np.abs(r - np.asarray(res)) <= 1e-10)
    D = (X.conj().T.contiguous() @ X - Y.conj().T.contiguous() @ Y).cpu().numpy()
    assert np.max(np.abs(D - np.diag(np.diag(D)))) < 1e-5
    s.close()


def test_timing_of_the_last_filter_after_a_failed_solve():
    # one Jacobi sweep does not converge in the first iteration: the solve ends
    # with CHASE_PH_ERR_EIG after its first filter, whose time and launches (two
    # products a degree) chase_ph_last_timing reports
    p = make_problem(300, lambda rng, m: rng.uniform(1.0, 5.0, m), 0.4, 12, 8, 10, 1e-10, seed=0)
    print_case("timing_after_failed_solve", m=p.m)
    A, B = dev_blocks(p)
    s = PHSolver(A, B, p.nev, p.nex, deg=10, rr_max_sweeps=1)
    with pytest.raises(ChasePHError) as e:
        s.solve(to_dev(p.w0_raw), to_dev(p.lanczos_raw))
    assert e.value.status == _lib.ERR_EIG
    ms, launches = s.last_timing()
    assert launches == 20
    assert 0 < ms < 1000
    s.apply_h(to_dev(p.w0_raw))
    assert s.last_timing()[1] == 1
    s.close()


def test_solve_projects_off_locked_pairs_on_wide_real_products():
    # With 168 of 600 pairs locked after four iterations the fifth one projects 864
    # columns of 8000 reals off 336: C = Qp^T X and X -= Qp C, both real and wide
    # enough for the 64 x 64 tiles (8000 x 864 >= 400 x 128 x 128 outputs, K = 336
    # beyond the short products).  A fault there would leave the new basis
    # non-orthogonal: every pair locked then against H V formed by matmul, and
    # eq. 3.5 between the old and the new ones
    m, nev, nex, tol = 4000, 560, 40, 1e-7
    print_case("solve_projection_wide_real", m=m, nev=nev, nex=nex)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)

    def normal(*shape):
        return torch.complex(torch.randn(shape, dtype=torch.float64, device="cuda", generator=gen),
                             torch.randn(shape, dtype=torch.float64, device="cuda", generator=gen))

    d = torch.linspace(1.0, 9.0, m, dtype=torch.float64, device="cuda")
    B = normal(m, m) * (0.05 / m ** 0.5)
    B = (0.5 * (B + B.T)).contiguous()
    A = torch.diag(d).to(torch.complex128)
    W0 = (torch.eye(2 * m, nev + nex, dtype=torch.complex128, device="cuda") + 1e-2 * normal(2 * m, nev + nex) / m ** 0.5)
    Lz = normal(2 * m, 4)
    locked = []
    for max_iter in (4, 5):
        s = PHSolver(A, B, nev, nex, deg=10, tol=tol, max_iter=max_iter, precision=FP64)
        ev, V, res, info = s.solve(W0.T.contiguous().T, Lz.T.contiguous().T, raise_on_noconv=False)
        locked.append(info.locked)
        s.close()
    before, now = locked
    cols = 2 * (nev + nex - before)
    assert 2 * m * cols >= 400 * 128 * 128 and 2 * m * cols * 2 * before > 2.8e8, locked
    assert now > before
    lam = torch.from_numpy(np.asarray(ev)[:now]).cuda().to(torch.complex128)
    V = V[:, :now]
    X, Y = V[:m], V[m:]
    HV = torch.cat([A @ X + B @ Y, -(B.conj() @ X) - A.conj() @ Y])
    r = torch.linalg.vector_norm(HV - V * lam[None, :], dim=0).cpu().numpy()
    assert np.all(r <= 1.5 * tol), r.max()
    assert np.all(np.abs(r - np.asarray(res)[:now]) <= 1e-10)
    D = (X.conj().T.contiguous() @ X - Y.conj().T.contiguous() @ Y).cpu().numpy()
    assert np.max(np.abs(D - np.diag(np.diag(D)))) < 1e-5
