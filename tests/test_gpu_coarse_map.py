"""The assembled coarse end of SPD hierarchies (all visits of a level below
its parent; the finest level too where the system is small) against the same
cycle level by level."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
amg = pytest.importorskip("paper_1503_01287_amd")
from paper_1503_01287_amd import problems

pytestmark = pytest.mark.gpu


def apply(s, r, k):
    b = torch.from_numpy(r).cuda()
    x = torch.zeros_like(b)
    if k == 1:
        s.precondition(b, x)
        return x
    B = torch.stack([b, 2 * b, -b])
    X = torch.zeros_like(B)
    s.solve_multi(B, X, tol=1e-10)
    return X.view(-1)


@pytest.mark.parametrize("nu,cycles", [(1, 1), (2, 1), (2, 2)])
@pytest.mark.parametrize("smoother", ["GS-1-1", "GS-2-1", "JA-1-1-0.5"])
@pytest.mark.parametrize("problem,n,first", [("laplace", 4, 0), ("elasticity", 4, 0), ("elasticity", 5, 1), ("laplace", 9, 1)])
def test_fused_equals_level_by_level(problem, n, first, smoother, nu, cycles):
    kw = dict(smoother=smoother, nu=nu, cycles=cycles, autotune=False)
    sysm = getattr(problems, problem)(n)
    fused = amg.AMGSolver(sysm, **kw)
    plain = amg.AMGSolver(sysm, fuse_coarse=False, **kw)
    assert [l for l in range(fused.num_levels) if fused.level_info(l).coarse_map] == [first]
    assert not any(plain.level_info(l).coarse_map for l in range(plain.num_levels))
    r = np.random.default_rng(n).standard_normal(sysm.dofs)
    # one linear map of at most a few thousand columns, each summed in
    # another order: as for the oracle's cycles, 1e-11; solves to 1e-10
    for k, tol in ((1, 1e-11), (3, 1e-8)):
        z, w = apply(fused, r, k), apply(plain, r, k)
        assert float((z - w).abs().max() / w.abs().max()) < tol, k


def test_reduced_cycles_with_several_visits_keep_their_levels():
    s = amg.AMGSolver(problems.elasticity(5), nu=2, precision="MIXED", krylov="FCG", autotune=False)
    assert not any(s.level_info(l).coarse_map for l in range(s.num_levels))
