"""GPU tests of the snapshots' FP64 check at the edges of its 16 x 16 tiles and
of the 64 snapshots: violation, objective, regularised and dual objective as
reported against the oracle's, recomputed from the returned potentials.

Both are FP64 sums over the same plan; its entries' exponents (a few hundred)
carry 1e-13 of rounding, and the entropy is a difference of sums about
|potential| / eps = 1e3 times larger: bars 1e-10 of the mass (violation) and 1e-9
relative (objectives)."""

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


@pytest.mark.parametrize("I,J,B", [(1, 1, 1), (15, 17, 2), (16, 16, 16), (64, 65, 17), (300, 33, 64), (1000, 15, 63),
                                   (2049, 130, 5), (33000, 20, 3), (130, 700, 9)])
def test_check_matches_the_oracle(A, oracle_lib, I, J, B):
    print(f"\n[case] snapshot check {I} x {J} x {B}", flush=True)
    rng = np.random.default_rng(I + J + B)
    C = rng.uniform(0.0, 1.0, (I, J)).astype(np.float32)
    a = rng.uniform(0.5, 1.5, (B, I))
    a /= a.sum(1, keepdims=True)
    b = rng.uniform(0.5, 1.5, J)
    b /= b.sum()
    eps = 0.05
    with A.Solver(I, J) as s:
        st, res = s.solve_snapshots(C, a, b, eps, 1e-4)
        assert st == A.OT_OK
        for q in sorted({0, B // 2, B - 1}):
            f, g = s.snapshot_potentials(q)
            chk = oracle_lib.plan_stats(C.astype(np.float64), a[q], b, f, g, eps)
            assert abs(res[q].marginal_violation - chk["marginal_violation"]) <= 1e-10
            for name in ("objective", "reg_objective", "dual_objective"):
                assert abs(getattr(res[q], name) - chk[name]) <= 1e-9 * max(abs(chk[name]), chk["objective"]), name
