"""GPU parity of phi = lambda ||x||_1 (+ box) and of the matrix-free Gram
operator Q = Ahat^T Ahat (the Lasso of Section 4.4, m = 0: the z -> x -> w
cycle of Remark 2.1) against the CPU oracle, through the C ABI.

Tolerances as for the CQP tests: operator 1e-13 relative; iterates over the
first 50 iterations 1e-10 of the largest entry; power method 1e-9; final
solutions both at relative KKT <= 1e-8 with objectives within 1e-6.
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


def _l1_box_csr():
    qp = qpgen.make_small_ccqp(seed=21, n=250, m=90, nb=40, density=0.05)
    qp.l1_weight = 0.8
    return qp


def _cases():
    return [qpgen.make_lasso(),
            qpgen.make_lasso(seed=77, p=777, q=3001, density=0.02),   # ragged sizes, p < q
            _l1_box_csr()]


def test_gram_operator_and_power_method():
    DP, Solver = _S()
    rng = np.random.default_rng(3)
    for qp in _cases()[:2]:
        s = Solver(DP(qp), power_start_Q=qpgen.power_start(qp.n), max_iter=1)
        x = rng.standard_normal(qp.n)
        Ah = qp.Ahat_scipy()
        assert _max_rel(s.apply("Q", x).cpu().numpy(), Ah.T @ (Ah @ x)) < 1e-13
        lq, _ = oracle.power(qp, "Q", qpgen.power_start(qp.n))
        assert s.power_info()["est_Q"] == pytest.approx(lq, rel=1e-9)
        s.close()


def test_iterates_match_oracle():
    DP, Solver = _S()
    K = 50
    for qp in _cases():
        lamQ = 1.01 * np.linalg.eigvalsh(qp.Q_dense()).max()
        lamA = 1.01 * np.linalg.eigvalsh(qp.A_scipy().toarray() @ qp.A_scipy().toarray().T).max() if qp.m else 0.0
        ro = oracle.solve(qp, tol=0.0, max_iter=K, check_every=10, lambda_A=lamA, lambda_Q=lamQ,
                          trace_iters=K, log_cap=K)
        s = Solver(DP(qp), lambda_A=lamA, lambda_Q=lamQ, tol=0.0, max_iter=K, check_every=10,
                   trace_iters=K, log_cap=K)
        rg = s.solve()
        s.close()
        np.testing.assert_array_equal(rg.check_log[:, 7], ro.check_log[:, 7])
        for col in (2, 3, 4, 5):
            np.testing.assert_allclose(rg.check_log[:, col], ro.check_log[:, col], rtol=1e-9, atol=1e-15)
        to = split_trace(ro.trace, qp.n, qp.m)
        tg = split_trace(rg.trace, qp.n, qp.m)
        for k in range(K):
            for name in ("y", "w", "x", "ybar", "wbar", "xbar"):
                if to[name].shape[1] == 0:
                    continue
                e = _max_rel(tg[name][k], to[name][k])
                assert e <= 1e-10, (k, name, e)


def test_full_solves_and_lasso_optimality():
    DP, Solver = _S()
    for qp in _cases():
        ro = oracle.solve(qp, tol=1e-8, max_iter=400_000)
        s = Solver(DP(qp), tol=1e-8, max_iter=400_000)
        rg = s.solve()
        s.close()
        assert rg.term == ro.term == "solved"
        assert rg.kkt <= 1e-8
        assert abs(rg.pobj - ro.pobj) <= 1e-6 * max(1.0, abs(ro.pobj))
        if qp.qkind == "gram":
            # subgradient optimality of the Lasso at the GPU's x
            x = rg.x.cpu().numpy()
            Ah, bh, lam = qp.Ahat_scipy(), qp.meta["bhat"], qp.l1_weight
            g = Ah.T @ (Ah @ x - bh)
            on = np.abs(x) > 1e-9 * max(1.0, np.abs(x).max())
            assert np.abs(g[on] + lam * np.sign(x[on])).max() <= 1e-5 * lam
            assert np.abs(g[~on]).max() <= lam * (1 + 1e-6)


def test_benchmark_size_kernels_match_oracle():
    """The benchmark's Lasso (p = 1e4, q = 5e5, 5e7 nonzeros) runs its Ahat x
    product on the column-split layout and Ahat^T t on the row-split kernel
    gathering from LDS by default: the Q operator against the oracle's, then
    three iterations with a check after each against the oracle.  lambda_Q is
    the host bound ||Ahat||_1 ||Ahat||_inf >= lambda_max(Ahat^T Ahat) on both
    sides (the power method would cost the oracle minutes here)."""
    import time
    DP, Solver = _S()
    t0 = time.time()
    qp = qpgen.make_lasso(seed=1006, p=10_000, q=500_000, density=0.01)
    Ah = qp.Ahat_scipy()
    lamQ = float(abs(Ah).sum(axis=0).max() * abs(Ah).sum(axis=1).max())
    print(f"lasso built ({time.time() - t0:.1f} s)", flush=True)
    dp = DP(qp)
    K = 3
    s = Solver(dp, lambda_Q=lamQ, tol=0.0, max_iter=K, check_every=1, log_cap=K)
    x = np.random.default_rng(4).standard_normal(qp.n)
    got = s.apply("Q", x).cpu().numpy()
    ref = oracle.apply_Q(qp, x)
    assert _max_rel(got, ref) < 1e-13
    rg = s.solve()
    s.close()
    print(f"gpu done ({time.time() - t0:.1f} s)", flush=True)
    ro = oracle.solve(qp, tol=0.0, max_iter=K, check_every=1, lambda_Q=lamQ, log_cap=K)
    print(f"oracle done ({time.time() - t0:.1f} s)", flush=True)
    np.testing.assert_allclose(rg.check_log[:, 2:6], ro.check_log[:, 2:6], rtol=1e-9, atol=1e-15)
    for name in ("w", "x", "z"):
        assert _max_rel(getattr(rg, name).cpu().numpy(), getattr(ro, name)) <= 1e-10, name


def test_batch_rejects_l1():
    from paper_2507_02470_amd.batch import BatchSolver
    from paper_2507_02470_amd._native import HPRQPError
    qp = qpgen.make_portfolio(3, n=60)
    qp.l1_weight = 0.1
    with pytest.raises(HPRQPError):
        BatchSolver([qp], tol=1e-8, max_iter=1000)


@pytest.mark.parametrize("rows,cols,avg,g", [(3, 40, 9, 1), (64, 300, 20, 2), (65, 300, 30, 8), (1000, 14336, 130, 16),
                                             (20_001, 700, 25, 4), (200, 9000, 700, 64), (66_000, 500, 40, 0)])
def test_row_split_products_from_lds(rows, cols, avg, g):
    """The row-split kernel over an LDS copy of the vector (16-bit columns, 64 rows a
    wave): every lane count, empty rows, rows past the eight entries a lane has in
    flight, a ragged last wave; g = 0 takes the default choice.  Bound: a sum of k
    products is off by at most (k + 1) u times their absolute sum."""
    import scipy.sparse as sp
    from paper_2507_02470_amd.solver import DeviceProblem, Solver
    rng = np.random.default_rng(rows)
    lens = rng.poisson(avg, rows)
    lens[rng.random(rows) < 0.1] = 0
    lens[rows // 3] = 10 * avg
    rp = np.concatenate([[0], np.cumsum(lens)])
    ci, v = rng.integers(0, cols, rp[-1]), rng.standard_normal(rp[-1])
    print(f"lds rows={rows} cols={cols} avg={avg} g={g}", flush=True)
    qp = qpgen.QP(n=cols, m=rows, qkind="zero", c=np.ones(cols), L=np.zeros(cols), U=np.ones(cols), a_rowptr=rp,
                  a_col=ci, a_val=v, l=np.zeros(rows), u=np.ones(rows))
    s = Solver(DeviceProblem(qp), lambda_A=1.0, tol=0.0, max_iter=1, spmv_lanes=-100 - g if g else -1)
    A, absA = (sp.csr_matrix((w, ci.copy(), rp.copy()), shape=(rows, cols)) for w in (v.copy(), np.abs(v)))
    x = rng.standard_normal(cols)
    got = s.apply("A", x).cpu().numpy()
    s.close()
    assert np.all(np.abs(got - A @ x) <= (lens + 1) * 2.0 ** -53 * (absA @ np.abs(x)) * 2.0)   # both sides round


@pytest.mark.parametrize("lens", [[1], [0, 1, 0], [2], [1, 2], [1, 1, 1], [0, 5, 0, 3, 1], [33, 0, 32, 1, 31, 64],
                                  [300, 1, 257, 0, 129, 1]])
@pytest.mark.parametrize("g", [1, 16, 64])
def test_row_split_products_read_entries_in_pairs(lens, g):
    """The row-split kernel over LDS reads pairs of entries that start at even
    positions: rows that begin or end inside a pair, a matrix of one entry, an odd
    number of entries (the last has no partner), entries past those in flight.
    Bound as above."""
    import scipy.sparse as sp
    from paper_2507_02470_amd.solver import DeviceProblem, Solver
    rows, cols = len(lens), 37
    rng = np.random.default_rng(sum(lens))
    rp = np.concatenate([[0], np.cumsum(lens)])
    ci, v = rng.integers(0, cols, rp[-1]), rng.standard_normal(rp[-1])
    print(f"pairs lens={lens} g={g}", flush=True)
    qp = qpgen.QP(n=cols, m=rows, qkind="zero", c=np.ones(cols), L=np.zeros(cols), U=np.ones(cols), a_rowptr=rp,
                  a_col=ci, a_val=v, l=np.zeros(rows), u=np.ones(rows))
    s = Solver(DeviceProblem(qp), lambda_A=1.0, tol=0.0, max_iter=1, spmv_lanes=-100 - g, small_path=0)
    A, absA = (sp.csr_matrix((w, ci.copy(), rp.copy()), shape=(rows, cols)) for w in (v.copy(), np.abs(v)))
    x = rng.standard_normal(cols)
    got = s.apply("A", x).cpu().numpy()
    s.close()
    assert np.all(np.abs(got - A @ x) <= (np.array(lens) + 1) * 2.0 ** -53 * (absA @ np.abs(x)) * 2.0)


@pytest.mark.parametrize("lanes", [-4, -3, -2, -116, 0, 1, 2, 64])
def test_iteration_in_either_form_for_every_product(lanes):
    """Without rows the step after Q xhat runs in the last product's epilogue where
    a thread there owns a row, else as a kernel of its own: the iterates of every
    product agree (sums in another order: 1e-10 relative, as between kernels
    elsewhere), over checks and restarts."""
    from paper_2507_02470_amd.solver import DeviceProblem, Solver
    qp = qpgen.make_lasso(seed=7, p=150, q=500)
    dp = DeviceProblem(qp)
    out = []
    for g in (4, lanes):
        s = Solver(dp, tol=0.0, max_iter=120, check_every=20, spmv_lanes=g, log_cap=20)
        r = s.solve()
        s.close()
        out.append(r)
    a, b = out
    np.testing.assert_array_equal(a.check_log[:, [0, 1, 7]], b.check_log[:, [0, 1, 7]])
    for k in ("x", "w", "z"):
        u, v = getattr(a, k).cpu().numpy(), getattr(b, k).cpu().numpy()
        assert np.max(np.abs(u - v)) <= 1e-10 * max(1.0, np.max(np.abs(u))), k


def test_columns_of_a_product_not_taken_are_given_back():
    """Autotuning times the row-split product over LDS, which reads 16-bit columns of its
    own: a handle that then runs another product holds no more memory than one
    that never timed it (each copy would be 24 MB here)."""
    from paper_2507_02470_amd.solver import DeviceProblem, Solver
    rng = np.random.default_rng(3)
    m, n, per = 12_000, 12_000, 1000
    rp = per * np.arange(m + 1)
    qp = qpgen.QP(n=n, m=m, qkind="zero", c=np.ones(n), L=np.zeros(n), U=np.ones(n), a_rowptr=rp,
                  a_col=rng.integers(0, n, rp[-1]), a_val=rng.standard_normal(rp[-1]), l=np.zeros(m), u=np.ones(m))
    dp = DeviceProblem(qp)
    used = []
    for tune in (0, 1, 0, 1):
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        s = Solver(dp, lambda_A=1.0, tol=0.0, max_iter=1, spmv_lanes=8, spmv_autotune=tune)
        torch.cuda.synchronize()
        used.append(free - torch.cuda.mem_get_info()[0])
        x = rng.standard_normal(n)
        y = s.apply("A", x)
        s.close()
    print("handle bytes", used, flush=True)
    assert bool(torch.isfinite(y).all())
    assert abs(used[3] - used[2]) < 12_000_000


@pytest.mark.parametrize("p,q,per_row", [(15_000, 700, 12), (15_000, 300, 200), (40_000, 64, 64)])
@pytest.mark.parametrize("m0_form", [-4, -3])
def test_iteration_in_the_epilogue_of_a_layout(p, q, per_row, m0_form):
    """As test_iteration_in_either_form_for_every_product, with an Ahat^T that has a
    column-split layout (more than 14,336 columns; panels of 16,384 and of 2,048) and a
    panel-ordered one: the iteration in the epilogue of those products."""
    from paper_2507_02470_amd.solver import DeviceProblem, Solver
    rng = np.random.default_rng(p + q)
    rp = per_row * np.arange(p + 1)
    ci = np.argsort(rng.random((p, q)), axis=1)[:, :per_row].ravel()
    v = rng.standard_normal(rp[-1]) / np.sqrt(p * per_row / q)
    none = dict(a_rowptr=np.zeros(1, np.int32), a_col=np.zeros(0, np.int32), a_val=np.zeros(0), l=np.zeros(0), u=np.zeros(0))
    qp = qpgen.QP(n=q, m=0, qkind="gram", c=rng.standard_normal(q), L=np.full(q, -np.inf), U=np.full(q, np.inf),
                  gram_p=p, gram_rowptr=rp, gram_col=ci, gram_val=v, l1_weight=0.1, **none)
    dp = DeviceProblem(qp)
    out = []
    for g in (4, m0_form):
        s = Solver(dp, tol=0.0, max_iter=120, check_every=20, spmv_lanes=g, log_cap=20)
        out.append(s.solve())
        s.close()
    a, b = out
    np.testing.assert_array_equal(a.check_log[:, [0, 1, 7]], b.check_log[:, [0, 1, 7]])
    for k in ("x", "w", "z"):
        u, w = getattr(a, k).cpu().numpy(), getattr(b, k).cpu().numpy()
        assert np.max(np.abs(u - w)) <= 1e-10 * max(1.0, np.max(np.abs(u))), k
