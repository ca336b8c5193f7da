"""GPU tests of which form a solve takes (sweeps, one cooperative launch with the
kernel in LDS, streamed from device memory, in FP64; teams in batches and
servers), and of the streamed form for every cost source and inside a caller's
workspace. Bars as for the other parity tests: violation < tol as reported and as
the oracle recomputes it; plans of two forms of one problem, each within the
residual bar of one solution, within 1e-6 in L1."""

import numpy as np
import pytest

import scenario as S

pytestmark = pytest.mark.gpu
EPS, TOL = 0.05, 1e-8


@pytest.fixture(scope="module")
def A():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1805_01559_amd import ot_assoc
    ot_assoc.lib()
    return ot_assoc


def uniform(I, J, seed):
    rng = np.random.default_rng(seed)
    a, b = rng.uniform(0.5, 1.5, I), rng.uniform(0.5, 1.5, J)
    return rng.uniform(0.1, 1.1, (I, J)), a / a.sum(), b / b.sum()


def problem(A, O, kind, I, J, host=True):
    """(solve(solver), FP64 cost, a, b) of one cost source."""
    if kind in ("geometry", "euclid"):
        L = S.make_layout(I, J, 1000.0, seed=I + J)
        if kind == "geometry":
            C, scale = O.cost(L)
            run = lambda s: s.solve_geometry(L.dev_xy, L.rrh_xy, L.radio, L.shadow_key, scale, L.a, L.b, EPS, TOL, 3000)
        else:
            d = L.dev_xy.astype(np.float64)[:, None, :] - L.rrh_xy.astype(np.float64)[None, :, :]
            C = np.sqrt((d**2).sum(2))
            scale = 2.0 * float(np.median(C))
            C /= scale
            run = lambda s: s.solve_euclid(L.dev_xy, L.rrh_xy, scale, L.a, L.b, EPS, TOL, 3000)
        return run, C, L.a, L.b
    C, a, b = uniform(I, J, I * J)
    dt = np.float64 if kind.endswith("64") else np.float32
    if kind.startswith("rates"):
        R = (1.0 / C).astype(dt)
        return (lambda s: s.solve_rates(R, 1.0, a, b, EPS, TOL, 3000)), 1.0 / R.astype(np.float64), a, b
    X = C.astype(dt)
    return (lambda s: s.solve_dense(X, a, b, EPS, TOL, 3000)), X.astype(np.float64), a, b


def solve(A, O, p, I, J, **opts):
    run, C, a, b = p
    with A.Solver(I, J, **opts) as s:
        st, res = run(s)
        f, g = s.potentials()
        form = A.ot_assoc_solve_form(s.h)
    chk = O.plan_stats(C, a, b, f, g, EPS)
    assert st == A.OT_OK and res.marginal_violation < TOL and chk["marginal_violation"] < TOL * 1.05
    assert bool(res.flags & A.OT_RESULT_PERSISTENT) == (form == A.OT_FORM_LDS)
    return form, O.plan(C, f, g, EPS)


@pytest.mark.parametrize("kind", ["dense32", "dense64", "rates32", "rates64", "euclid", "geometry"])
def test_form_by_cost_source(A, oracle_lib, kind):
    print(f"\n[case] forms of a {kind} cost", flush=True)
    lds = A.OT_FORM_SWEEPS if kind in ("dense64", "rates64") else A.OT_FORM_LDS
    for I, J, want in ((120, 25, lds), (3000, 130, lds),
                       (40003, 250, A.OT_FORM_STREAMED if lds == A.OT_FORM_LDS else A.OT_FORM_SWEEPS)):
        p = problem(A, oracle_lib, kind, I, J)
        form, P = solve(A, oracle_lib, p, I, J)
        assert form == want
        form, P0 = solve(A, oracle_lib, p, I, J, persistent=0)
        assert form == A.OT_FORM_SWEEPS
        assert np.abs(P - P0).sum() <= 1e-6


def test_form_in_fp64(A, oracle_lib):
    print("\n[case] forms in FP64 precision", flush=True)
    F = A.OT_PREC_FP64
    for kind, I, J, want in (("dense64", 90, 20, 3), ("dense32", 2999, 197, 3), ("geometry", 2000, 130, 3),
                             ("rates64", 900, 70, 0), ("euclid", 900, 70, 0), ("dense64", 20001, 250, 0),
                             ("dense64", 300, 1025, 0)):
        p = problem(A, oracle_lib, kind, I, J)
        assert solve(A, oracle_lib, p, I, J, precision=F)[0] == want, (kind, I, J)
        assert solve(A, oracle_lib, p, I, J, precision=F, persistent=0)[0] == A.OT_FORM_SWEEPS


@pytest.mark.parametrize("kind", ["dense32", "geometry", "euclid", "rates32"])
def test_streamed_within_a_workspace(A, oracle_lib, kind):
    """Room beyond the fixed buffers holds the staged host matrix or the kept
    FP64 cost, and the streamed kernel behind it."""
    import torch
    I, J = 40003, 250
    print(f"\n[case] streamed {kind} in a workspace", flush=True)
    p = problem(A, oracle_lib, kind, I, J)
    n = A.ot_assoc_workspace_size(I, J)
    first = {"dense32": 4, "rates32": 4, "geometry": 8, "euclid": 0}[kind] * I * J
    ker = 4 * I * 252
    ws = torch.empty(n + first + 256 + ker, dtype=torch.uint8, device="cuda")
    plans = []
    for size, want in ((n + first + 256 + ker, A.OT_FORM_STREAMED), (n + first + ker - 256, A.OT_FORM_SWEEPS),
                       (n + first, A.OT_FORM_SWEEPS)):
        n0 = A.ot_assoc_device_allocations()
        form, P = solve(A, oracle_lib, p, I, J, workspace=ws.data_ptr(), workspace_bytes=size)
        assert form == want and A.ot_assoc_device_allocations() == n0
        plans.append(P)
    assert max(np.abs(P - plans[0]).sum() for P in plans) <= 1e-6


def test_teams_are_what_ran(A, oracle_lib):
    print("\n[case] instances solved by teams", flush=True)
    xs = [uniform(I, J, I) for I, J in ((80, 20), (3000, 130), (6000, 400), (70, 512), (30000, 400))]
    args = [[x[0].astype(np.float32) for x in xs], [x[1] for x in xs], [x[2] for x in xs]]
    for opts, teams in ((dict(), 4), (dict(persistent=0), 0)):
        with A.Solver(16, 16, batch_tune=0, **opts) as s:
            st, res = s.solve_batch(*args, EPS, TOL)
            assert st == A.OT_OK and all(r.marginal_violation < TOL for r in res)
            assert A.ot_assoc_batch_teams(s.h) == teams
    with A.Server() as srv:
        for x in zip(*args):
            srv.submit(*x, EPS, TOL)
        n = 0
        while n < len(xs):
            done = srv.progress()
            assert all(c.result.status == A.OT_OK for c in done)
            n += len(done)
        assert A.ot_serve_teams(srv.s) == 4
