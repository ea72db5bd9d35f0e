"""What an isolated solve leaves in a plan ends with the next set-up of another
geometry: products that would read its pair matrix with the atoms of that
geometry are refused."""
import numpy as np
import pytest

from inputs import gen

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def T(a):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")


# fewer, as many and more atoms than the isolated system had
@pytest.mark.parametrize("n", [40, 64, 200])
def test_descriptors_end_an_isolated_solve(n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2607_17978_amd import qeq
    s = gen.cluster_system(n, q_tot=0.0, seed=3)
    d = gen.system_64()
    args = (T(s.pos), T(s.sigma), T(s.J), T(s.chi), s.q_tot)
    species = torch.as_tensor(s.species, dtype=torch.int32, device="cuda")
    plan = qeq.Plan(200, tol=1e-8, max_iter=2000)
    q = plan.solve_nonperiodic(*args)[0]
    pots = plan.element_potentials(species, 2)
    plan.descriptors(T(d.pos), d.cell, T(d.sigma), np.linspace(1.0, 8.0, 8), 1.0, 8.0)
    with pytest.raises(qeq.QEqError) as e:
        plan.element_potentials(torch.zeros(d.n, dtype=torch.int32, device="cuda"), 2)
    assert e.value.code == qeq.QEQ_EINVAL
    with pytest.raises(qeq.QEqError):
        plan.time_kernel(len(qeq.Plan.PROFILE_KINDS))
    # and the next isolated solve brings them back
    assert torch.equal(plan.solve_nonperiodic(*args)[0], q)
    assert torch.equal(plan.element_potentials(species, 2), pots)
    plan.close()
