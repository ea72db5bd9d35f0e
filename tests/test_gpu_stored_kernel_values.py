"""The isolated solve's products from stored kernel values.

At the solution (E + diag J) q + chi is the same for every atom.  The sum is
formed here in FP64 with plain torch at the solver's own charges, so what is
left is the solve's residual and the FP32 rounding of the kernel values K_ij:
about six roundings each (distance, width, their product, erf, quotient), bounded
by 8 ulp of every term.  Sizes sit on the edges of the 64-atom tiles, with odd
and even tile counts, and where the splits of the sum change.
"""
import math

import numpy as np
import pytest

from inputs import gen

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 63, 64, 65, 129, 257, 1000, 4097, 8193])
def test_stationary_in_64_bits(n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2607_17978_amd import qeq
    s = gen.cluster_system(n, q_tot=1.0, seed=n)
    d = {k: torch.as_tensor(np.ascontiguousarray(getattr(s, k)), dtype=torch.float64, device="cuda")
         for k in ("pos", "sigma", "J", "chi")}
    plan = qeq.Plan(n, tol=1e-8, max_iter=3000)
    q, _, _, st = plan.solve_nonperiodic(d["pos"], d["sigma"], d["J"], d["chi"], s.q_tot)
    species = torch.as_tensor(s.species, dtype=torch.int32, device="cuda")
    pots = plan.element_potentials(species, 2)
    plan.close()
    assert st["rc"] == 0
    eq, mag, part = (torch.empty(n, dtype=torch.float64, device="cuda") for _ in range(3))
    for a in range(0, n, 1024):
        b = min(n, a + 1024)
        r = torch.cdist(d["pos"][a:b], d["pos"], compute_mode="donot_use_mm_for_euclid_dist")
        at = torch.arange(a, b, device="cuda")
        r[at - a, at] = 1e30
        g = torch.sqrt(d["sigma"][a:b, None] ** 2 + d["sigma"][None, :] ** 2)
        K = torch.erf(r / (math.sqrt(2.0) * g)) / r
        eq[a:b] = K @ q
        mag[a:b] = K @ q.abs()
        part[a:b] = K @ (q * (species == 0))
    ulp = 8.0 * 2.0 ** -24
    grad = eq + q / (d["sigma"] * math.sqrt(math.pi)) + d["J"] * q + d["chi"]
    dev = grad - grad.mean()
    chi_norm = float((d["chi"] - d["chi"].mean()).norm())
    assert float(dev.norm()) <= ulp * float(mag.norm()) + 2e-7 * chi_norm
    # the element products read the same values
    assert bool(((pots[:, 0] - part).abs() <= ulp * mag + 1e-12).all())
