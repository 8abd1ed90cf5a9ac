"""The assembled coarse map of a Vanka cycle stays off where its assembly would
cost many solves (16^3: 1,388 columns)."""
import pytest

torch = pytest.importorskip("torch")
amg = pytest.importorskip("paper_1503_01287_amd")
from paper_1503_01287_amd import problems

pytestmark = pytest.mark.gpu


def test_no_map_that_a_solve_does_not_pay_for():
    s = problems.mixed_elasticity(16)
    solver = amg.AMGSolver(s, smoother="Vanka-1-1", krylov="FGMRES")
    assert not any(solver.level_info(l).fused for l in range(solver.num_levels))
    b = torch.from_numpy(s.rhs).cuda()
    x = torch.zeros_like(b)
    assert solver.solve(b, x, tol=1e-8).converged


def test_a_map_that_it_pays_for():
    s = problems.mixed_elasticity(5)
    solver = amg.AMGSolver(s, smoother="Vanka-1-1", krylov="FGMRES")
    assert [solver.level_info(l).fused for l in range(solver.num_levels)] == [0, 1, 1]
