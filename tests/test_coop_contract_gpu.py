"""GPU tests of what the interface promises of solves, batches and servers,
where one cooperative launch does the work that sweeps did: refused inputs,
options, limits and memory."""

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


def instance(I, J, seed, mass=1.0):
    rng = np.random.default_rng(seed)
    C = rng.uniform(0.0, 1.0, (I, J)).astype(np.float32)
    a, b = rng.uniform(0.5, 1.5, I), rng.uniform(0.5, 1.5, J)
    return C, mass * a / a.sum(), mass * b / b.sum()


def serve(srv, n, limit=20000):
    done = []
    for _ in range(limit):
        done += srv.progress()
        if len(done) >= n:
            return sorted(done, key=lambda c: c.user_tag)
    raise AssertionError("server did not finish")


@pytest.mark.parametrize("I,J", [(300, 20), (2000, 60), (1500, 400)])
@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
def test_non_finite_cost_ends_a_batched_instance(A, I, J, bad):
    """A single forbidden link, which alone would leave the problem solvable."""
    print(f"\n[case] batch and server, {bad} among the costs of {I} x {J}", flush=True)
    good, x = instance(500, 30, 1), instance(I, J, 2)
    x[0][I // 2, J - 1] = bad
    for tol in (1e-6, 1e-9):
        with A.Solver(16, 16, batch_tune=0) as s, pytest.raises(A.OTError, match="numerically"):
            s.solve_batch([good[0], x[0]], [good[1], x[1]], [good[2], x[2]], 0.05, tol, 500)
        with A.Server() as srv:
            for k, y in enumerate((good, x)):
                srv.submit(*y, 0.05, tol, 500, user_tag=k)
            assert [c.result.status for c in serve(srv, 2)] == [A.OT_OK, A.OT_ENUMERIC]


@pytest.mark.parametrize("I,J,off", [(700, 33, 25), (1500, 200, 27), (3000, 400, 20), (2000, 700, 25)])
def test_fp32_noise_of_plain_sums_with_column_offsets(A, oracle_lib, I, J, off):
    """check_every holds the phase at its fixed point for dozens of iterations
    of FP32 sums. Their noise is three roundings of a row (entry, scaling, sum)
    of 2^-24 at most and 2.1e-8 in the mean, 3.6e-8 together, the first two
    averaged over the row; columns average over hundreds of rows: bar 4e-8."""
    print(f"\n[case] FP32 noise {I} x {J}, column offsets of {off} eps", flush=True)
    rng, eps = np.random.default_rng(I), 0.01
    C = (rng.uniform(0.0, 0.05, (I, J)) + np.linspace(0.0, off * eps, J)).astype(np.float32)
    _, a, b = instance(I, J, J)
    with A.Solver(I, J, check_every=48) as s:
        st, res = s.solve_dense(C, a, b, eps, 4e-7, 400)
        f, g = s.potentials()
    assert st == A.OT_OK and (res.iterations, res.fp64_iterations) == (48, 0)
    chk = oracle_lib.plan_stats(C.astype(np.float64), a, b, f, g, eps)
    assert res.marginal_violation < 4e-8 and chk["marginal_violation"] < 4e-8


@pytest.mark.parametrize("I,J", [(150, 20), (2000, 60), (3000, 400), (1200, 1100)])
def test_polish_iters_act(A, I, J):
    """polish_iters FP64 iterations end a solve below the FP32 noise, and none
    one that met a tol above it. They are the FP64 iteration applied to the
    unpolished potentials: exponents of up to 30 carry 4e-15 of rounding, the
    exchanged sums 2^-51; bar 1e-12 per iteration in units of eps."""
    print(f"\n[case] polish_iters {I} x {J}", flush=True)
    C, a, b = instance(I, J, 3)
    C64, eps, tol = C.astype(np.float64), 0.05, 1e-9
    got = []
    for n in (0, 1, 3):
        with A.Solver(I, J, polish_iters=n) as s:
            assert s.solve_dense(C, a, b, eps, 1e-6)[1].fp64_iterations == 0
            st, res = s.solve_dense(C, a, b, eps, tol)
            f, g = s.potentials()
            assert st == A.OT_OK and res.flags & A.OT_RESULT_PERSISTENT
            assert res.fp64_iterations == n
            got.append((res.iterations, f, g))
            if n:
                st, res = s.solve_dense(C, a, b, eps, tol, max_iter=got[0][0] + 1)
                assert st == A.OT_OK and (res.iterations, res.fp64_iterations) == (got[0][0] + 1, 1)
    assert [x[0] - got[0][0] for x in got] == [0, 1, 3]
    lse = lambda x, axis: x.max(axis) + np.log(np.exp(x - np.expand_dims(x.max(axis), axis)).sum(axis))
    g = got[0][2]
    for k in range(1, 4):
        f = eps * (np.log(a) - lse((g - C64) / eps, 1))
        g = eps * (np.log(b) - lse((f[:, None] - C64) / eps, 0))
        for n, fn, gn in got[1:]:
            if n == got[0][0] + k:
                assert np.abs(fn - f).max() <= 1e-12 * k * eps and np.abs(gn - g).max() <= 1e-12 * k * eps
    if J <= 512:
        for n in (0, 1, 3):
            with A.Solver(16, 16, batch_tune=0, polish_iters=n) as s, A.Server(polish_iters=n) as srv:
                assert s.solve_batch([C], [a], [b], eps, 1e-6)[1][0].fp64_iterations == 0
                srv.submit(C, a, b, eps, tol)
                for res in (s.solve_batch([C], [a], [b], eps, tol)[1][0], serve(srv, 1)[0].result):
                    assert res.fp64_iterations == n and res.marginal_violation < tol


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_refused_matrix_in_sweeps_writes_no_plan(A, dtype):
    import torch
    print(f"\n[case] refused matrix in sweeps, {dtype.__name__}", flush=True)
    C, a, b = instance(900, 60, 5)
    C[3, 4] = np.inf
    prec = A.OT_PREC_FP32 if dtype == np.float32 else A.OT_PREC_FP64
    with A.Solver(900, 60, persistent=0, precision=prec) as s:
        plan = torch.full((900, 60), -7.0, device="cuda")
        s.set_plan_output(plan)
        with pytest.raises(A.OTError, match="non-finite"):
            s.solve_dense(C.astype(dtype), a, b, 0.05, 1e-8)
        assert bool((plan == -7.0).all())


@pytest.mark.parametrize("I,J", [(100, 20), (4000, 60), (75001, 128)])
@pytest.mark.parametrize("kind", ["rates", "dense", "dense64"])
def test_refused_matrix_ends_the_solve_at_once(A, I, J, kind):
    """A negative rate or an infinite cost makes no NaN: the verdict itself has
    to end the solve, which would go on for minutes here (2e7 iterations), and
    nothing may be written."""
    import time
    import torch
    print(f"\n[case] refused {kind} matrix {I} x {J}", flush=True)
    C, a, b = instance(I, J, 4)
    X = (1.0 / (C + np.float32(0.1))) if kind == "rates" else C
    X[I - 1, J // 2] = -1.0 if kind == "rates" else np.inf
    f64 = kind == "dense64"
    with A.Solver(I, J, precision=A.OT_PREC_FP64 if f64 else A.OT_PREC_FP32) as s:
        solve = (lambda *x: s.solve_rates(X, 1.0, *x)) if kind == "rates" else (lambda *x: s.solve_dense(X, *x))
        if f64:
            X = X.astype(np.float64)
        plan = torch.full((I, J), -7.0, device="cuda")
        s.set_plan_output(plan)
        n = 200_000 if f64 and I > 50000 else 20_000_000  # (the first sweeps make the check where no launch does)
        t = time.time()
        with pytest.raises(A.OTError, match="not finite and positive" if kind == "rates" else "non-finite"):
            solve(a, b, 0.05, 1e-300, n)
        assert time.time() - t < 5.0
        assert bool((plan == -7.0).all())


@pytest.mark.parametrize("mass", [1e-34, 3e-30, 1e-20, 0.7, 1e20, 1e33])
@pytest.mark.parametrize("I,J", [(150, 20), (2000, 60)])
def test_total_mass_far_from_one(A, I, J, mass):
    """Marginals in another unit: the same iterations (scalings by a power of
    two are exact; by the factors here the marginals round anew, so that a
    residual may land on the other side of tol once) and the same potentials,
    f shifted by eps ln(mass). Column offsets of 25 eps make the row sums
    drift over 2^30 between references."""
    print(f"\n[case] total mass {mass:g}, {I} x {J}", flush=True)
    rng, eps = np.random.default_rng(6), 0.01
    C = (rng.uniform(0.0, 0.05, (I, J)) + np.linspace(0.0, 25 * eps, J)).astype(np.float32)
    _, a, b = instance(I, J, 6)
    for tol in (1e-5, 1e-9):
        with A.Solver(I, J) as s, A.Solver(16, 16, batch_tune=0) as sb:
            _, ref = s.solve_dense(C, a, b, eps, tol)
            st, res = s.solve_dense(C, mass * a, mass * b, eps, tol)
            stb, (rb,) = sb.solve_batch([C], [mass * a], [mass * b], eps, tol)
        for q, r in ((st, res), (stb, rb)):
            assert q == A.OT_OK and r.marginal_violation < tol and abs(r.iterations - ref.iterations) <= 1
            assert abs(r.objective / mass - ref.objective) <= 4 * tol * C.max()


def test_progress_runs_a_bounded_share(A, oracle_lib):
    """One progress call runs 64 iterations of what is in flight at most: a
    request that needs hundreds is still running after the first call, one that
    arrives then and needs few finishes before it, and the slow one ends as it
    does alone, bit for bit."""
    print("\n[case] a fast request overtakes a slow one", flush=True)
    L = S.make_layout(700, 60, 2000.0, hot_spots=2, hot_share=0.4, seed=78)
    d = L.dev_xy.astype(np.float64)[:, None, :] - L.rrh_xy.astype(np.float64)[None, :, :]
    C = np.sqrt((d**2).sum(2))
    C = (C / np.median(C)).astype(np.float32)
    eps = 0.02
    got = []
    for fast in (False, True):
        for tol in (1e-6, 1e-9):
            order = []
            with A.Server() as srv:
                srv.submit(C, L.a, L.b, eps, tol, 20000, layout_key=1, user_tag=0)
                calls = 1
                order += srv.progress()
                assert not order and srv.counts()[1] == 1
                if fast:
                    srv.submit(*instance(900, 70, 5), 0.05, 1e-6, 2000, user_tag=1)
                while len(order) < 1 + fast:
                    order += srv.progress()
                    calls += 1
                f, g = srv.potentials(1, 700, 60)
            if fast:
                assert order[0].user_tag == 1 and order[0].result.status == A.OT_OK
            res = order[-1].result
            assert res.status == A.OT_OK and res.iterations > 250 and calls >= res.iterations / 64
            chk = oracle_lib.plan_stats(C.astype(np.float64), L.a, L.b, f, g, eps)
            assert res.marginal_violation < tol and chk["marginal_violation"] < tol * 1.05
            got.append((f, g, res.iterations))
    for x, y in zip(got[:2], got[2:]):
        assert x[2] == y[2] and np.array_equal(x[0], y[0]) and np.array_equal(x[1], y[1])


def test_a_long_polish_is_shared_out_too(A):
    """150 FP64 iterations end a request over several progress calls, and one in
    a batch in one call; both are what the option asks for."""
    print("\n[case] polish_iters 150 in a server and a batch", flush=True)
    x = instance(900, 70, 5)
    with A.Server(polish_iters=150) as srv:
        srv.submit(*x, 0.05, 1e-8, 2000)
        calls, done = 1, srv.progress()
        assert not done and srv.counts()[1] == 1
        while not done:
            done = srv.progress()
            calls += 1
        a = done[0].result
        assert A.ot_serve_teams(srv.s) == 1
    with A.Solver(16, 16, batch_tune=0, polish_iters=150) as s:
        b = s.solve_batch(*([y] for y in x), 0.05, 1e-8, 2000)[1][0]
    assert a.status == b.status == A.OT_OK and calls >= 3
    assert a.fp64_iterations == b.fp64_iterations == 150 and a.iterations == b.iterations


def slot_bytes(I, J):
    """A server request's own device memory: padded FP32 cost, marginals, two
    sets of potentials, sweep partials of 64 rows, each part 256-byte aligned."""
    up = lambda x: (x + 255) // 256 * 256
    parts = (I + 63) // 64
    return (up(4 * I * ((J + 3) // 4 * 4)) + 3 * up(8 * I) + 3 * up(8 * J) + up(8 * parts * J) + up(8 * parts) +
            up(40 * parts) + 256)


def test_team_memory_counts_in_the_budget(A):
    """The exchange block of a request's team is part of what it holds, and a
    request whose budget has no room for one is solved all the same."""
    print("\n[case] exchange blocks within the server's budget", flush=True)
    I, J = 3100, 130
    C, a, b = instance(I, J, 8)
    stage, own = 4 * I * J, slot_bytes(I, J)
    with A.Server() as srv:
        srv.submit(C, a, b, 0.002, 1e-300, 100000)
        srv.progress()
        assert srv.counts()[1] == 1 and srv.counts()[3] >= own + 2 * 8 * 8 * 512  # (replicas of v alone)
        n0 = A.ot_assoc_device_allocations()
        for _ in range(3):
            srv.progress()
        assert A.ot_assoc_device_allocations() == n0
    tight = float(own + (stage + 255) // 256 * 256)
    for budget, st in ((tight, A.OT_OK), (tight - 256, A.OT_ENOMEM)):
        with A.Server(budget_bytes=budget) as srv:
            for k in range(2):
                srv.submit(C, a, b, 0.05, 1e-8, user_tag=k)
            done = serve(srv, 2)
            assert [c.result.status for c in done] == [st, st] and A.ot_serve_teams(srv.s) == 0
            assert srv.counts()[3] == 0


def test_batch_wait_that_gives_up(A):
    """Scalings withheld at the third iteration: every team ends by giving up,
    the error says so, and the next batch on the handle runs as usual."""
    print("\n[case] teams whose waits give up", flush=True)
    xs = [instance(I, J, I) for I, J in ((200, 20), (3000, 60), (6000, 300))]
    args = [[x[q] for x in xs] for q in range(3)]
    with A.Solver(16, 16, batch_tune=0) as s:
        assert A.ot_assoc_test_hold_exchange(3) == A.OT_OK
        with pytest.raises(A.OTError, match="gave up") as e:
            s.solve_batch(*args, 0.05, 1e-8)
        assert e.value.status == A.OT_EDEVICE
        st, res = s.solve_batch(*args, 0.05, 1e-8)
        assert st == A.OT_OK and all(r.marginal_violation < 1e-8 for r in res)


def test_batch_of_several_launches(A):
    """More instances than one launch takes (1024), and instances whose teams
    would keep one launch too long: the same results as alone, bit for bit."""
    import torch
    print("\n[case] batches of several team launches", flush=True)
    for n, I, J, picks in ((1100, 120, 20, (0, 1023, 1024, 1099)), (400, 8000, 400, (0, 170, 399))):
        C, a, b = (torch.from_numpy(x).cuda() for x in instance(I, J, 11))
        eps = np.linspace(0.05, 0.08, n)
        with A.Solver(16, 16, batch_tune=0) as s:
            st, res = s.solve_batch([C] * n, [a] * n, [b] * n, eps, 1e-6)
            assert st == A.OT_OK and all(r.marginal_violation < 1e-6 for r in res)
            got = [s.batch_potentials(k) for k in picks]
        with A.Solver(16, 16, batch_tune=0) as s:
            for k, (f, g) in zip(picks, got):
                s.solve_batch([C], [a], [b], [eps[k]], 1e-6)
                f1, g1 = s.batch_potentials(0)
                assert np.array_equal(f, f1) and np.array_equal(g, g1)


def test_solver_batch_and_server_in_threads(A):
    """Cooperative launches of three handles, each on its own stream and thread:
    the same results as one after the other, bit for bit."""
    import threading
    import torch
    print("\n[case] solver, batch and server side by side", flush=True)
    xs = [tuple(torch.from_numpy(x).cuda() for x in instance(I, J, I)) for I, J in ((9000, 300), (700, 40), (3000, 130))]

    def single(n):
        with A.Solver(9000, 300) as s:
            for _ in range(n):
                st, res = s.solve_dense(*xs[0], 0.05, 1e-8)
                assert st == A.OT_OK
            return s.potentials()

    def batch(n):
        with A.Solver(16, 16, batch_tune=0) as s:
            for _ in range(n):
                st, _ = s.solve_batch(*([x[q] for x in xs] for q in range(3)), 0.05, 1e-8)
                assert st == A.OT_OK and A.ot_assoc_batch_teams(s.h) == 3
            return sum((s.batch_potentials(k) for k in range(3)), ())

    def server(n):
        with A.Server() as srv:
            for k in range(n):
                for x in xs[:2]:
                    srv.submit(*x, 0.05, 1e-8, 2000)
                srv.submit(*xs[2], 0.05, 1e-8, 2000, layout_key=k + 1)
                assert all(c.result.status == A.OT_OK for c in serve(srv, 3))
            return srv.potentials(n, 3000, 130)

    jobs = (single, batch, server)
    want = [job(1) for job in jobs]
    got = [None] * 3
    torch.cuda.synchronize()

    def work(k):
        try:
            got[k] = jobs[k](40)
        except Exception as e:  # (reported by the comparison below)
            got[k] = e

    threads = [threading.Thread(target=work, args=(k,)) for k in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for x, y in zip(want, got):
        assert not isinstance(y, Exception), y
        assert all(np.array_equal(p, q) for p, q in zip(x, y))
