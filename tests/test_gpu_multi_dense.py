"""Blocks of right-hand sides against the same systems one by one: the first
iterations, which show the fused vector passes, and the coarse end's dense map
at sizes off its tiles."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
amg = pytest.importorskip("paper_1503_01287_amd")
from paper_1503_01287_amd import problems

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,krylov", [("FP64", "PCG"), ("FP64", "FCG"), ("FP32", "FCG"), ("MIXED", "FCG"), ("MIXED", "PCG")])
@pytest.mark.parametrize("problem,n", [("laplace", 5), ("laplace", 9), ("elasticity", 5), ("elasticity", 8)])
def test_iterations_equal_one_by_one(problem, n, precision, krylov):
    sysm = getattr(problems, problem)(n)
    s = amg.AMGSolver(sysm, smoother="GS-1-1", krylov=krylov, precision=precision, autotune=False)
    assert any(s.level_info(l).coarse_map for l in range(s.num_levels))
    rng = np.random.default_rng(n)
    # sums of the same terms in another order: a few hundred roundings of the
    # cycle's precision, carried through two or three further iterations
    bound = 4096 * (2.0 ** -53 if precision == "FP64" else 2.0 ** -24)
    for k in (1, 2, 3, 5, 8):
        B = torch.from_numpy(rng.standard_normal((k, sysm.dofs))).cuda()
        for steps in (1, 2, 4):
            X = torch.zeros_like(B)
            s.solve_multi(B, X, tol=1e-30, maxit=steps)
            for r in range(k):
                x = torch.zeros_like(B[r])
                s.solve(B[r], x, tol=1e-30, maxit=steps)
                assert float((X[r] - x).norm() / x.norm()) < bound, (k, steps, r)
