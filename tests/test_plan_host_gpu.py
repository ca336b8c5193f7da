"""GPU test of plans to host memory: whole, in blocks of the staging (a plan
above 64 MB) and through the work region of a caller's workspace, bit for bit
the plan written to device memory."""

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


@pytest.mark.parametrize("I,J,dtype", [(3, 2, np.float32), (1000, 50, np.float32), (1000, 50, np.float64),
                                       (31001, 300, np.float64)])
def test_host_plan_is_the_device_plan(A, I, J, dtype):
    import torch
    print(f"\n[case] host plan {I} x {J} {dtype.__name__}", flush=True)
    rng = np.random.default_rng(I)
    C = rng.uniform(0.0, 1.0, (I, J)).astype(np.float32)
    a, b = rng.uniform(0.5, 1.5, I), rng.uniform(0.5, 1.5, J)
    a, b = a / a.sum(), b / b.sum()
    with A.Solver(I, J) as s:
        for _ in range(2):  # (the staging is the solve's scratch: solve, plan, solve, plan)
            st, _ = s.solve_dense(C, a, b, 0.05, 1e-7)
            assert st == A.OT_OK
            host = s.plan(dtype=dtype)
            dev = torch.empty((I, J), dtype=torch.float32 if dtype == np.float32 else torch.float64, device="cuda")
            s.plan(dev)
            assert np.array_equal(host, dev.cpu().numpy())
