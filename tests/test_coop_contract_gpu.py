"""GPU tests of what the interface promises of solves, batches and servers,
where one cooperative launch does the work that sweeps did: refused inputs,
options, limits and memory."""

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
