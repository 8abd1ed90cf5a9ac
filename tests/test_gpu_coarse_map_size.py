"""From which level the cycle is one assembled map: with several visits of a
level only up to the sizes whose assembly a solve pays for."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
amg = pytest.importorskip("paper_1503_01287_amd")
from paper_1503_01287_amd import problems

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,smoother,nu,first,unknowns", [
    (9, "GS-2-2", 2, 1, 2940), (10, "GS-2-2", 2, 2, 4113), (10, "GS-2-2", 1, 1, 4113),
    (7, "JA-1-1-0.5", 2, 1, 1452), (8, "JA-1-1-0.5", 2, None, 2211), (8, "JA-1-1-0.5", 1, 1, 2211)])
def test_first_level_of_the_map(n, smoother, nu, first, unknowns):
    s = problems.elasticity(n)
    kw = dict(smoother=smoother, nu=nu, autotune=False)
    fused, plain = amg.AMGSolver(s, **kw), amg.AMGSolver(s, fuse_coarse=False, **kw)
    assert fused.level_dofs(1) == unknowns
    assert [l for l in range(fused.num_levels) if fused.level_info(l).coarse_map] == ([] if first is None else [first])
    r = torch.from_numpy(np.random.default_rng(n).standard_normal(s.dofs)).cuda()
    z, w = torch.zeros_like(r), torch.zeros_like(r)
    fused.precondition(r, z)
    plain.precondition(r, w)
    # the same sums in another order, at most some 4000 terms
    assert float((z - w).abs().max() / w.abs().max()) < 1e-11
