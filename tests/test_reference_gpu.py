"""GPU tests of the stabilised kernel's references in the cooperative phase and
of the FP64 geometry cost a solve keeps: where a reference has to be renewed
(scalings that leave the FP32 range, long delta phases), the widths at which
the kernel instantiations change, and geometry costs kept in memory against
costs regenerated in every pass (a handle on a workspace without room for
them). Bars as for the other parity tests: violation < tol as reported and as
the oracle recomputes it, transport cost within 1e-6 relative and the plan
within 1e-6 in L1 of the oracle's converged solution."""

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


def check(O, C, a, b, eps, tol, f, g, res):
    ref = O.sinkhorn(C, a, b, eps, 1e-12, 60000)
    chk, rst = O.plan_stats(C, a, b, f, g, eps), O.plan_stats(C, a, b, ref.f, ref.g, eps)
    assert res.marginal_violation < tol and chk["marginal_violation"] < tol * 1.05
    assert abs(chk["objective"] - rst["objective"]) <= 1e-6 * abs(rst["objective"])
    assert np.abs(O.plan(C, f, g, eps) - O.plan(C, ref.f, ref.g, eps)).sum() <= 1e-6
    return ref


def marginals(rng, I, J):
    a, b = rng.uniform(0.5, 1.5, I), rng.uniform(0.5, 1.5, J)
    return a / a.sum(), b / b.sum()


@pytest.mark.parametrize("I,J", [(33, 32), (700, 33), (300, 416), (300, 417), (257, 512), (129, 1024), (65, 1025)])
@pytest.mark.parametrize("tol", [1e-5, 1e-8, 1e-10])
def test_column_offsets_renew_the_reference(A, oracle_lib, I, J, tol):
    """Costs with a per-column offset of up to 50 eps: the first scalings span
    2^72, past the range in which a plain reference is kept (2^40)."""
    print(f"\n[case] column offsets {I}x{J} tol {tol}", flush=True)
    rng = np.random.default_rng(1000 * I + J)
    eps = 0.01
    C = (rng.uniform(0.0, 0.05, (I, J)) + np.linspace(0.0, 50 * eps, J)).astype(np.float32)
    a, b = marginals(rng, I, J)
    with A.Solver(I, J) as s:
        st, res = s.solve_dense(C, a, b, eps, tol, 5000)
        f, g = s.potentials()
    assert st == A.OT_OK and res.flags & A.OT_RESULT_PERSISTENT
    C64 = C.astype(np.float64)
    if tol > 1e-7:  # the plan is that far from the converged one: only what tol promises
        assert oracle_lib.plan_stats(C64, a, b, f, g, eps)["marginal_violation"] < tol * 1.05
    else:
        check(oracle_lib, C64, a, b, eps, tol, f, g, res)


def test_slow_convergence_in_delta_sums(A, oracle_lib):
    """A distance cost that takes hundreds of iterations below the FP32 noise:
    they run as delta sums of renewed FP64 references, not as FP64 sweeps."""
    print("\n[case] distance cost 1500x60, slow convergence", flush=True)
    L = S.make_layout(1500, 60, 2000.0, hot_spots=2, hot_share=0.4, seed=77)
    d = L.dev_xy.astype(np.float64)[:, None, :] - L.rrh_xy.astype(np.float64)[None, :, :]
    C = np.sqrt((d**2).sum(2))
    scale = float(np.median(C))
    C /= scale
    with A.Solver(1500, 60) as s:
        st, res = s.solve_euclid(L.dev_xy, L.rrh_xy, scale, L.a, L.b, 0.02, 1e-9, 20000)
        f, g = s.potentials()
    assert st == A.OT_OK and res.flags & A.OT_RESULT_PERSISTENT
    ref = oracle_lib.sinkhorn(C, L.a, L.b, 0.02, 1e-9, 60000)
    assert abs(res.iterations - ref.iters) <= 8 and res.fp64_iterations <= 8
    check(oracle_lib, C, L.a, L.b, 0.02, 1e-9, f, g, res)


@pytest.mark.parametrize("I,J", [(70, 1), (130, 64), (131, 65), (90, 512), (67, 513), (41, 1025), (30, 2048)])
def test_geometry_kept_and_regenerated(A, oracle_lib, I, J):
    """The same geometry solve on a handle that keeps the FP64 cost and on one
    whose workspace has no room for it."""
    import torch
    print(f"\n[case] geometry {I}x{J}, kept and regenerated", flush=True)
    L = S.make_layout(I, J, 1000.0, seed=31 * I + J)
    C, scale = oracle_lib.cost(L)
    eps, tol = 0.05, 1e-8
    n = A.ot_assoc_workspace_size(I, J)
    room = torch.empty(n + 8 * I * J, dtype=torch.uint8, device="cuda")
    for size in (None, n, n + 8 * I * J):
        opts = {} if size is None else dict(workspace=room.data_ptr(), workspace_bytes=size)
        with A.Solver(I, J, **opts) as s:
            st, res = s.solve_geometry(L.dev_xy, L.rrh_xy, L.radio, L.shadow_key, scale, L.a, L.b, eps, tol, 5000)
            f, g = s.potentials()
            P = s.plan()
        assert st == A.OT_OK
        check(oracle_lib, C, L.a, L.b, eps, tol, f, g, res)
        P0 = oracle_lib.plan(C, f, g, eps)
        assert np.abs(P - P0).max() <= 1e-9 * P0.max()  # (the same FP64 cost up to its rounding, times 1 / eps)


@pytest.mark.parametrize("I,J", [(75001, 128), (40003, 250), (20481, 400), (10005, 1000), (5201, 2045)])
def test_streamed_kernel_above_the_lds(A, oracle_lib, I, J):
    """Instances whose kernel does not fit in LDS: held in device memory when
    there is room, else (a workspace without any) the chunked sweeps."""
    import torch
    print(f"\n[case] streamed kernel {I}x{J}", flush=True)
    rng = np.random.default_rng(I + J)
    C = rng.uniform(0.0, 1.0, (I, J)).astype(np.float32)
    a, b = marginals(rng, I, J)
    eps, tol = 0.05, 1e-8
    Cd, ad, bd = (torch.from_numpy(x).cuda() for x in (C, a, b))
    n = A.ot_assoc_workspace_size(I, J)
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")
    plans = []
    for opts in ({}, dict(workspace=ws.data_ptr(), workspace_bytes=n)):
        with A.Solver(I, J, **opts) as s:
            st, res = s.solve_dense(Cd, ad, bd, eps, tol, 3000)
            f, g = s.potentials()
        assert st == A.OT_OK and not res.flags & A.OT_RESULT_PERSISTENT
        C64 = C.astype(np.float64)
        chk = oracle_lib.plan_stats(C64, a, b, f, g, eps)
        assert res.marginal_violation < tol and chk["marginal_violation"] < tol * 1.05
        plans.append(oracle_lib.plan(C64, f, g, eps))
    # both within the residual bar of one solution
    assert np.abs(plans[0] - plans[1]).sum() <= 1e-6
