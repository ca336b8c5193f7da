"""GPU tests of the teams that solve a batch's instances (one launch, each
instance on as many workgroups as its kernel needs LDS for): sizes at the
edges of the column classes and of one workgroup, instances too large for the
LDS of the GPU, an iteration cap that a slow instance reaches (it goes on in
sweeps), and bitwise independence of the rest of the batch. Bars as for the
other batch tests: violation < tol as reported and as the oracle recomputes
it, the plan within 1e-6 in L1 of the oracle's converged one."""

import numpy as np
import pytest

import scenario as S

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def A():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1805_01559_amd import ot_assoc
    ot_assoc.lib()
    return ot_assoc


def instance(I, J, seed):
    rng = np.random.default_rng(seed)
    a, b = rng.uniform(0.5, 1.5, I), rng.uniform(0.5, 1.5, J)
    return rng.uniform(0.0, 1.0, (I, J)).astype(np.float32), a / a.sum(), b / b.sum()


def check(O, x, f, g, res, eps, tol):
    C, (a, b) = x[0].astype(np.float64), x[1:]
    chk = O.plan_stats(C, a, b, f, g, eps)
    assert res.marginal_violation < tol and chk["marginal_violation"] < tol * 1.05
    assert abs(res.objective - chk["objective"]) <= 1e-9 * abs(chk["objective"])
    ref = O.sinkhorn(C, a, b, eps, 1e-12, 60000)
    assert np.abs(O.plan(C, f, g, eps) - O.plan(C, ref.f, ref.g, eps)).sum() <= max(1e-6, 20 * tol)


SIZES = [(1, 1), (17, 32), (300, 33), (1100, 128), (270, 129), (290, 256), (150, 257), (64, 416), (130, 417), (70, 512),
         (1153, 31), (20481, 400)]


@pytest.mark.parametrize("tol", [1e-6, 1e-9])
def test_team_sizes(A, oracle_lib, tol):
    eps = 0.05
    xs = [instance(I, J, 100 * I + J) for I, J in SIZES]
    print(f"\n[case] teams over {SIZES}, tol {tol}", flush=True)
    with A.Solver(16, 16, batch_tune=0) as s:
        st, res = s.solve_batch([x[0] for x in xs], [x[1] for x in xs], [x[2] for x in xs], eps, tol, 3000)
        assert st == A.OT_OK, [r.status for r in res]
        pots = [s.batch_potentials(k) for k in range(len(xs))]
        pick = [3, 8, 0]
        st, _ = s.solve_batch([xs[k][0] for k in pick], [xs[k][1] for k in pick], [xs[k][2] for k in pick], eps, tol,
                              3000)
        for q, k in enumerate(pick):
            f, g = s.batch_potentials(q)
            assert np.array_equal(f, pots[k][0]) and np.array_equal(g, pots[k][1])
    for k, x in enumerate(xs):
        check(oracle_lib, x, *pots[k], res[k], eps, tol)


def test_team_iteration_cap_and_sweeps_after_it(A, oracle_lib):
    """A distance cost that needs more iterations than one team launch runs
    (1024 in a batch, 256 in a server) next to one that does not."""
    print("\n[case] slow instance past the team launch's cap", flush=True)
    L = S.make_layout(700, 60, 2000.0, hot_spots=2, hot_share=0.4, seed=78)
    d = L.dev_xy.astype(np.float64)[:, None, :] - L.rrh_xy.astype(np.float64)[None, :, :]
    C = np.sqrt((d**2).sum(2))
    slow = ((C / np.median(C)).astype(np.float32), L.a, L.b)
    fast = instance(900, 70, 5)
    eps, tol = [0.005, 0.05], 1e-7
    ref = oracle_lib.sinkhorn(slow[0].astype(np.float64), L.a, L.b, eps[0], tol, 60000)
    assert ref.iters > 1100
    xs = [slow, fast]
    with A.Solver(16, 16, batch_tune=0) as s:
        st, res = s.solve_batch([x[0] for x in xs], [x[1] for x in xs], [x[2] for x in xs], eps, tol, 60000)
        assert st == A.OT_OK
        got = [s.batch_potentials(k) for k in range(2)]
    with A.Server() as srv:
        for k, x in enumerate(xs):
            srv.submit(x[0], x[1], x[2], eps[k], tol, 60000, layout_key=k + 1, user_tag=k)
        done = []
        while len(done) < 2:
            done += srv.progress()
        assert all(c.result.status == A.OT_OK for c in done)
        got += [srv.potentials(k + 1, *xs[k][0].shape) for k in range(2)]
        res = list(res) + [c.result for c in sorted(done, key=lambda c: c.user_tag)]
    for q, (f, g) in enumerate(got):
        x = xs[q % 2]
        chk = oracle_lib.plan_stats(x[0].astype(np.float64), x[1], x[2], f, g, eps[q % 2])
        assert res[q].marginal_violation < tol and chk["marginal_violation"] < tol * 1.05
