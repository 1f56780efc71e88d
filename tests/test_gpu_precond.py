"""GPU parity of the diagonal preconditioning (Section 4.1: Ruiz passes, then
Pock-Chambolle with alpha = 1, explicit Q; termination on the given problem)
against the CPU oracle, through the C ABI.

Tolerances: scale factors 1e-13 relative (same products and sums, different
rounding order at most); iterates over the first 50 iterations and final
solutions as in the unpreconditioned tests (1e-10 of the largest entry;
objective 1e-6 relative).
"""
import numpy as np
import pytest

import oracle
import qpgen
from oracle.oracle import split_trace

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2507_02470_amd import load
    load()


def _S():
    from paper_2507_02470_amd.solver import DeviceProblem, Solver
    return DeviceProblem, Solver


def _max_rel(a, b):
    return np.max(np.abs(a - b)) / max(1.0, np.max(np.abs(b)))


def _badly_scaled(qp, seed):
    """The same QP with variables and rows rescaled by 10^U(-2, 2)."""
    rng = np.random.default_rng(seed)
    Q, A = qp.Q_dense(), qp.A_scipy().toarray()
    s = 10.0 ** rng.uniform(-2, 2, qp.n)
    r = 10.0 ** rng.uniform(-2, 2, qp.m)
    return qpgen.from_dense(s[:, None] * Q * s[None, :], s * qp.c, qp.L / s, qp.U / s,
                            r[:, None] * A * s[None, :], r * qp.l, r * qp.u)


def _scaled_lams(qp, D, E):
    """lambda's of the scaled problem (dense), from the oracle's scale factors."""
    Q, A = qp.Q_dense(), qp.A_scipy().toarray()
    As = E[:, None] * A * D[None, :]
    Qs = D[:, None] * Q * D[None, :]
    lamA = 1.01 * np.linalg.eigvalsh(As @ As.T).max() if qp.m else 0.0
    lamQ = 1.01 * np.linalg.eigvalsh(Qs).max()
    return lamA, lamQ


def _cases():
    return [_badly_scaled(qpgen.make_small_ccqp(), 3),
            _badly_scaled(qpgen.make_small_ccqp(seed=7, n=300, m=140, nb=60, density=0.04), 4)]


def test_scale_factors_match_oracle():
    DP, Solver = _S()
    for qp in _cases():
        for ruiz in (0, 1, 10):
            D0, E0 = oracle.scaling(qp, ruiz_iters=ruiz)
            s = Solver(DP(qp), precondition=1, ruiz_iters=ruiz, max_iter=1)
            D, E = s.scaling()
            s.close()
            assert _max_rel(D.cpu().numpy(), D0) < 1e-13
            assert _max_rel(E.cpu().numpy(), E0) < 1e-13


def test_preconditioned_iterates_match_oracle():
    DP, Solver = _S()
    K = 50
    for qp in _cases():
        D0, E0 = oracle.scaling(qp)
        lamA, lamQ = _scaled_lams(qp, D0, E0)
        ro = oracle.solve(qp, tol=0.0, max_iter=K, check_every=10, lambda_A=lamA, lambda_Q=lamQ,
                          trace_iters=K, log_cap=K, precondition=True)
        s = Solver(DP(qp), lambda_A=lamA, lambda_Q=lamQ, tol=0.0, max_iter=K, check_every=10,
                   trace_iters=K, log_cap=K, precondition=1)
        rg = s.solve()
        s.close()
        np.testing.assert_array_equal(rg.check_log[:, 7], ro.check_log[:, 7])
        for col in (2, 3, 4, 5):   # R, eta_p, eta_d, eta_gap of the given problem
            np.testing.assert_allclose(rg.check_log[:, col], ro.check_log[:, col], rtol=1e-9, atol=1e-15)
        to = split_trace(ro.trace, qp.n, qp.m)
        tg = split_trace(rg.trace, qp.n, qp.m)
        for k in range(K):
            for name in ("y", "w", "x", "ybar", "wbar", "xbar"):
                e = _max_rel(tg[name][k], to[name][k])
                assert e <= 1e-10, (k, name, e)
        for name in ("y", "z", "w", "x"):
            assert _max_rel(getattr(rg, name).cpu().numpy(), getattr(ro, name)) <= 1e-10, name


def test_preconditioned_full_solve_and_given_problem_entry_points():
    DP, Solver = _S()
    qp = _cases()[0]
    ro = oracle.solve(qp, tol=1e-8, max_iter=400_000, precondition=True)
    s = Solver(DP(qp), tol=1e-8, max_iter=400_000, precondition=1)
    rg = s.solve()
    assert rg.term == ro.term == "solved"
    assert rg.kkt <= 1e-8
    assert abs(rg.pobj - ro.pobj) <= 1e-6 * max(1.0, abs(ro.pobj))
    # the returned point is in the given variables: the given problem's
    # residuals (oracle, CPU) agree with what the solver reported
    res = oracle.residuals(qp, rg.y.cpu().numpy(), rg.z.cpu().numpy(), rg.x.cpu().numpy())
    assert res["kkt"] <= 1e-8
    for k in ("eta_p", "eta_d", "eta_gap"):
        assert getattr(rg, k) == pytest.approx(res[k], rel=1e-6, abs=1e-14)
    # hprqp_residuals and hprqp_apply act on the given problem
    # (the eta's are normalised differences of O(1) sums over n terms: at 1e-9 they
    # carry an absolute rounding of a few 1e-15 up to ~1e-14 on either side)
    g = s.residuals(rg.y, rg.z, rg.x)
    for k in ("eta_p", "eta_d", "eta_gap", "pobj", "dobj"):
        assert g[k] == pytest.approx(res[k], rel=1e-9, abs=1e-13), k
    rng = np.random.default_rng(1)
    x = rng.standard_normal(qp.n); y = rng.standard_normal(qp.m)
    A = qp.A_scipy()
    assert _max_rel(s.apply("A", x).cpu().numpy(), A @ x) < 1e-13
    assert _max_rel(s.apply("AT", y).cpu().numpy(), A.T @ y) < 1e-13
    assert _max_rel(s.apply("Q", x).cpu().numpy(), qp.Q_dense() @ x) < 1e-13
    # a warm start in the given variables from the solution stops at the first check
    s.set_options(max_iter=400_000)
    rw = s.solve(y0=rg.y, w0=rg.w, x0=rg.x)
    assert rw.term == "solved" and rw.iters <= 100
    s.close()
    # the badly scaled QP is a change of variables of the well-scaled one: same
    # optimal value (the badly scaled one is not solved in 4e5 iterations
    # without preconditioning)
    r0 = oracle.solve(qpgen.make_small_ccqp(), tol=1e-8, max_iter=400_000)
    assert abs(rg.pobj - r0.pobj) <= 1e-6 * max(1.0, abs(r0.pobj))


def test_matrix_free_q_ignores_preconditioning():
    DP, Solver = _S()
    qp = qpgen.make_portfolio(12, n=300)
    s0 = Solver(DP(qp), tol=1e-8, max_iter=100_000)
    s1 = Solver(DP(qp), tol=1e-8, max_iter=100_000, precondition=1)
    D, E = s1.scaling()
    assert torch.all(D == 1.0) and torch.all(E == 1.0)
    r0, r1 = s0.solve(), s1.solve()
    assert r0.iters == r1.iters
    assert torch.equal(r0.x, r1.x)
    s0.close(); s1.close()


@pytest.mark.parametrize("scale,start", [(1.0, "ones"), (1e60, "ones"), (1e-60, "ones"), (1e10, "hidden"), (1e25, "hidden")])
def test_power_method_over_scales_and_starts(scale, start):
    """The power method keeps its vector unnormalized over a chunk of iterations:
    matrices of extreme scale, and a start almost orthogonal to the dominant
    direction (the chunk overflows and is taken again step by step), give the
    estimate and count of the method as stated, written out here.  A diagonal A
    makes every step exact up to roundings: 3 u a step and entry, n u a sum."""
    from paper_2507_02470_amd.solver import DeviceProblem, Solver
    n = 64
    rng = np.random.default_rng(9)
    a = np.sqrt(scale) * rng.uniform(0.5, 1.0, n)
    v0 = np.ones(n)
    if start == "hidden":
        a[:] = rng.uniform(0.5, 1.0, n)
        a[5] = scale
        v0[5] = 1e-3 / scale ** 2
    rows = np.arange(n + 1)
    qp = qpgen.QP(n=n, m=n, qkind="zero", c=np.ones(n), L=np.zeros(n), U=np.ones(n), a_rowptr=rows,
                  a_col=np.arange(n), a_val=a, l=np.zeros(n), u=np.ones(n))
    print(f"power method scale={scale} start={start}", flush=True)
    s = Solver(DeviceProblem(qp), power_start_A=v0, tol=0.0, max_iter=1)
    info = s.power_info()
    s.close()
    v = v0 / np.linalg.norm(v0)
    lam = 0.0
    for it in range(1, 5001):
        w = a * (a * v)
        new = v @ w
        stop = it > 1 and abs(new - lam) <= 1e-6 * abs(new)
        lam, v = new, w / np.linalg.norm(w)
        if stop:
            break
    assert info["it_A"] == it
    assert abs(info["est_A"] - lam) <= 2 * (6 * it + 2 * n + 10) * 2.0 ** -53 * lam


def test_chunk_that_overflows_leaves_nothing_for_a_solve_without_rows():
    """A chunk of the power method that overflows leaves infinities in the
    reduction slots; without rows a solve never writes some of them, and reads
    them as 0: the same result as with lambda_Q given (a run of its own, with no
    power method)."""
    from paper_2507_02470_amd.solver import DeviceProblem, Solver
    n, big = 64, 1e30
    q = np.random.default_rng(2).uniform(0.5, 1.0, n)
    q[5] = big
    v0 = np.ones(n)
    v0[5] = 1e-3 / big
    qp = qpgen.QP(n=n, m=0, qkind="csr", c=np.linspace(-1.0, 1.0, n), L=np.full(n, -2.0), U=np.full(n, 2.0),
                  a_rowptr=np.zeros(1, np.int32), a_col=np.zeros(0, np.int32), a_val=np.zeros(0),
                  l=np.zeros(0), u=np.zeros(0), q_rowptr=np.arange(n + 1, dtype=np.int32),
                  q_col=np.arange(n, dtype=np.int32), q_val=q)
    for small in (0, 1):
        kw = dict(tol=0.0, max_iter=60, check_every=20, small_path=small, sigma0=1.0)
        s = Solver(DeviceProblem(qp), power_start_Q=v0, **kw)
        a = s.solve()
        s.close()
        assert a.lambda_Q == pytest.approx(1.01 * big, rel=1e-12)
        s = Solver(DeviceProblem(qp), lambda_Q=a.lambda_Q, **kw)
        b = s.solve()
        s.close()
        print("small_path", small, a.term, a.sigma, b.term, b.sigma, flush=True)
        assert a.term == b.term and a.iters == b.iters and a.sigma == b.sigma
        assert np.isfinite(a.sigma)
        for k in ("x", "w", "z"):
            assert torch.equal(getattr(a, k), getattr(b, k)), k


@pytest.mark.parametrize("kind", ["gram", "csr", "csr_small", "zero"])
def test_estimates_leave_nothing_in_the_slots_of_a_solve(kind):
    """The power method uses the reduction slots of an iteration; a solve without
    rows, or with Q = 0, never writes some of them and reads them as 0.  A solve
    that takes its own estimates equals, to the last bit and over its restarts,
    one that is given the same lambdas."""
    import scipy.sparse as sp
    from paper_2507_02470_amd.solver import DeviceProblem, Solver
    rng = np.random.default_rng(11)
    n, i32 = 400, np.int32
    none = dict(a_rowptr=np.zeros(1, i32), a_col=np.zeros(0, i32), a_val=np.zeros(0), l=np.zeros(0), u=np.zeros(0))
    if kind == "gram":
        qp = qpgen.make_lasso(seed=3, p=60, q=n)
    elif kind == "zero":
        qp = qpgen.make_tiny(5, n=8, m=4, qkind="zero")
    else:
        B = sp.random(n, n, 0.02, random_state=rng, data_rvs=rng.standard_normal)
        Q = (B @ B.T + 0.01 * sp.eye(n)).tocsr()
        Q.sort_indices()
        qp = qpgen.QP(n=n, m=0, qkind="csr", c=rng.standard_normal(n), L=np.full(n, -2.0), U=np.full(n, 2.0),
                      q_rowptr=Q.indptr.astype(i32), q_col=Q.indices.astype(i32), q_val=Q.data, **none)
    kw = dict(tol=0.0, max_iter=600, check_every=20, log_cap=100, sigma0=1.0, small_path=int(kind == "csr_small"))
    if kind == "gram":
        kw.pop("small_path")
    dp = DeviceProblem(qp)
    s = Solver(dp, **kw)
    a = s.solve()
    s.close()
    lam = dict(lambda_Q=a.lambda_Q) if qp.qkind != "zero" else {}
    if qp.m:
        lam["lambda_A"] = a.lambda_A
    s = Solver(dp, **lam, **kw)
    b = s.solve()
    s.close()
    assert a.restarts > 1
    np.testing.assert_array_equal(a.check_log, b.check_log)
    for k in ("x", "w", "z"):
        assert torch.equal(getattr(a, k), getattr(b, k)), k
