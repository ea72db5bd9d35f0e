"""qeq_batched_last_ms counts the kernels of a call, not the preparation on the host."""
import time

import numpy as np
import pytest

from inputs import gen

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def T(a):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")


def args(cells):
    d = gen.system_64()
    m = len(cells)
    return dict(pos=T(np.tile(d.pos, (m, 1))), offsets=[64 * k for k in range(m + 1)], cells=np.stack(cells),
                sigma=T(np.tile(d.sigma, m)), J=T(np.tile(d.J, m)), chi=T(np.tile(d.chi, m)), q_tot=[0.0] * m)


def test_no_kernel_no_time():
    """Structures that are all refused on the host launch nothing."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2607_17978_amd import qeq
    d = gen.system_64()
    plan = qeq.Plan(64)
    rc = plan.solve_batched(**args([np.zeros((3, 3))] * 8))[4]
    assert rc == qeq.QEQ_EINVAL and plan.batched_ms() == 0.0
    # and one that is solved counts no more than the call takes
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    rc = plan.solve_batched(**args([np.zeros((3, 3)), d.cell]))[4]
    wall = (time.perf_counter() - t0) * 1e3
    assert rc == qeq.QEQ_EINVAL and 0.0 < plan.batched_ms() <= wall
    assert plan.batched_ms() == 0.0
    plan.close()
