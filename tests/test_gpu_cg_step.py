"""The one-block CG step (at most 2,048 atoms) at the edges of its block sizes.

The solve's charges must sum to the total and leave the gradient E q + J q +
chi constant, measured with the operator product on its own: the tolerance
1e-6 on the relative residual, doubled where the solve may stop restarting.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 63, 255, 256, 257, 511, 512, 513, 1023, 1024, 1025, 2047, 2048, 2049])
def test_step_edges(n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2607_17978_amd import qeq
    rng = np.random.default_rng([81, n])
    L = max(12.0, (n / 0.01) ** (1.0 / 3.0))
    cell = np.diag([L, L, L])
    side = int(np.ceil(n ** (1.0 / 3.0)))
    sites = np.stack(np.meshgrid(*[np.arange(side)] * 3, indexing="ij"), -1).reshape(-1, 3)[rng.permutation(side ** 3)[:n]]
    T = lambda a: torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")
    pos = T((sites + 0.5 + rng.uniform(-0.2, 0.2, (n, 3))) * (L / side))
    sigma, J, chi = T(rng.uniform(1.0, 1.6, n)), T(rng.uniform(0.3, 0.6, n)), T(rng.normal(0.0, 0.1, n))
    plan = qeq.Plan(n, eta=2.0, r_cut=11.0, tol=1e-6)
    q, _, _, st = plan.solve(pos, cell, sigma, J, chi, 0.0)
    g = plan.matvec(pos, cell, sigma, q) + J * q + chi
    plan.close()
    assert st["rc"] == 0
    assert abs(float(q.sum())) <= 1e-9 * max(1.0, float(q.abs().sum()))
    ref = float((chi - chi.mean()).norm())
    assert float((g - g.mean()).norm()) <= 2e-6 * max(ref, 1e-30)
