"""CG with the cycle replayed as a graph or launched kernel by kernel, whichever
the handle's cycle calls for: the same kernels in the same order, hence the
same bits as with graphs off."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
amg = pytest.importorskip("paper_1503_01287_amd")
from paper_1503_01287_amd import problems

pytestmark = pytest.mark.gpu

CASES = {  # both answers of the rule, for both smoothers and precisions
    "Gauss-Seidel, mapped": dict(n=6, smoother="GS-1-1"),
    "Gauss-Seidel, level by level": dict(n=5, smoother="GS-2-1", fuse_coarse=False),
    "Gauss-Seidel W, reduced": dict(n=5, smoother="GS-1-1", nu=2, precision="MIXED"),
    "Gauss-Seidel by colour": dict(n=5, smoother="GS-1-1", by_colour=True),
    "Gauss-Seidel by colour, reduced": dict(n=5, smoother="GS-1-1", by_colour=True, precision="FP32"),
    "Jacobi, mapped": dict(n=6, smoother="JA-1-1-0.5"),
    "Jacobi, whole": dict(n=3, smoother="JA-2-1-0.5"),
    "Jacobi, level by level": dict(n=5, smoother="JA-1-1-0.5", fuse_coarse=False),
    "Jacobi, two levels, reduced": dict(n=3, smoother="JA-1-1-0.5", precision="MIXED"),
    "Jacobi W, mapped at 1": dict(n=7, smoother="JA-1-1-0.5", nu=2),
    "Jacobi W, reduced": dict(n=7, smoother="JA-1-1-0.5", nu=2, precision="MIXED"),
    "one level": dict(n=2, smoother="JA-1-1-0.5", max_levels=1),
}


@pytest.mark.parametrize("case", list(CASES))
@pytest.mark.parametrize("krylov", ["PCG", "FCG"])
def test_same_bits(case, krylov):
    kw = dict(CASES[case])
    n, by_colour = kw.pop("n"), kw.pop("by_colour", False)
    sysm = problems.elasticity(n)
    pair = [amg.AMGSolver(sysm, krylov=krylov, autotune=False, graph=g, **kw) for g in (True, False)]
    for s in pair:
        for l in range(s.num_levels - 1 if by_colour else 0):
            s.set_launch_shape(l, "sweep" if kw.get("precision", "FP64") == "FP64" else "sweep_rp", 32)
    rng = np.random.default_rng(n)
    for k in range(4):
        b = torch.from_numpy(sysm.rhs if k == 0 else rng.standard_normal(sysm.dofs)).cuda()
        got = []
        for s in pair:
            x = torch.zeros_like(b)
            r = s.solve(b, x, tol=1e-9, maxit=4 if k == 3 else 200)
            got.append((x, r.iters, r.status, r.relres))
        assert torch.equal(got[0][0], got[1][0]) and got[0][1:] == got[1][1:], k
