"""GPU tests of the cooperative phase in FP64 against the FP64 sweeps
(persistent=0) and the oracle: column-class edges, one workgroup and many, a
cost so wide that the reference is renewed, warm starts, the iteration limit
and a tol below the phase's range.

Both paths compute the same iterates, so iteration counts are equal and the
plans differ by rounding only: exponents of up to a few hundred carry 1e-14
of absolute rounding, the fixed-point map amplifies it by 1 / (1 - rate),
below 1000 here; the bar is 1e-11 in L1 (plan mass 1)."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def A():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1805_01559_amd import ot_assoc
    ot_assoc.lib()
    return ot_assoc


def instance(I, J, seed, width=1.0):
    rng = np.random.default_rng(seed)
    a, b = rng.uniform(0.5, 1.5, I), rng.uniform(0.5, 1.5, J)
    return width * rng.uniform(0.0, 1.0, (I, J)), a / a.sum(), b / b.sum()


def solve(A, x, eps, tol, iters=4000, coop=1, dtype=np.float64, warm=None):
    C, a, b = x
    with A.Solver(*C.shape, precision=A.OT_PREC_FP64, persistent=coop) as s:
        out = []
        for a_q in ([a] if warm is None else [a, warm]):
            st, res = s.solve_dense(C.astype(dtype), a_q, b, eps, tol, iters, warm_start=len(out) > 0)
            f, g = s.potentials()
            out.append((st, res, f, g, s.plan(dtype=np.float64)))
        return out


def same(x, y):
    assert x[0] == y[0] and x[1].iterations == y[1].iterations
    assert x[1].fp64_iterations == y[1].fp64_iterations and x[1].flags == y[1].flags == 0
    assert np.abs(x[4] - y[4]).sum() <= 1e-11
    assert abs(x[1].objective - y[1].objective) <= 1e-11 * abs(y[1].objective)


SIZES = [(1, 1), (40, 64), (900, 65), (2999, 128), (4099, 129), (513, 256), (2050, 257), (20000, 31), (3333, 416),
         (417, 417), (5000, 512), (1025, 513), (2500, 1024), (1200, 1025)]


@pytest.mark.parametrize("I,J", SIZES)
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_sizes(A, oracle_lib, I, J, dtype):
    print(f"\n[case] FP64 phase {I} x {J} {dtype.__name__}", flush=True)
    x = instance(I, J, I + J)
    x = (x[0].astype(dtype).astype(np.float64), x[1], x[2])
    eps, tol = 0.05, 1e-10
    got, ref = solve(A, x, eps, tol, dtype=dtype)[0], solve(A, x, eps, tol, coop=0, dtype=dtype)[0]
    same(got, ref)
    assert got[0] == A.OT_OK and got[1].marginal_violation < tol
    chk = oracle_lib.plan_stats(x[0], x[1], x[2], got[2], got[3], eps)
    assert chk["marginal_violation"] < tol * 1.01 and abs(got[1].objective - chk["objective"]) <= 1e-11


@pytest.mark.parametrize("I,J,width,eps", [(700, 60, 1.0, 0.003), (1500, 200, 4.0, 0.05), (300, 20, 1.0, 0.002)])
def test_reference_renewed(A, I, J, width, eps):
    """A device far from every RRH but one sends its scaling past 2^40 within a
    few iterations; the reference is then taken anew."""
    print(f"\n[case] FP64 phase, wide cost {I} x {J}", flush=True)
    x = instance(I, J, 7, width)
    x[0][:, : J // 2] += 0.5 * width  # half of the columns start far below their share
    got, ref = solve(A, x, eps, 1e-9, 600)[0], solve(A, x, eps, 1e-9, 600, coop=0)[0]
    same(got, ref)
    assert np.ptp(got[3]) / eps > 40 * np.log(2.0)


def test_warm_start_limit_and_tight_tol(A):
    print("\n[case] FP64 phase: warm start, iteration limit, tight tol", flush=True)
    x = instance(1700, 90, 3)
    a2 = x[1] * np.random.default_rng(4).uniform(0.99, 1.01, 1700)
    a2 /= a2.sum()
    for warm in (a2, x[1]):  # (with unchanged marginals the start is within tol already)
        for p, q in zip(solve(A, x, 0.05, 1e-9, warm=warm), solve(A, x, 0.05, 1e-9, warm=warm, coop=0)):
            same(p, q)
    got, ref = solve(A, x, 0.05, 1e-10, 5)[0], solve(A, x, 0.05, 1e-10, 5, coop=0)[0]
    same(got, ref)
    assert got[0] == A.OT_WARN_MAXITER
    same(solve(A, x, 0.05, 1e-14, 300)[0], solve(A, x, 0.05, 1e-14, 300, coop=0)[0])


def test_bad_cost_is_refused(A):
    x = instance(500, 40, 9)
    x[0][311, 17] = np.nan
    with A.Solver(500, 40, precision=A.OT_PREC_FP64) as s:
        with pytest.raises(A.OTError):
            s.solve_dense(x[0], x[1], x[2], 0.05, 1e-8)
