"""CG iterations replayed as graphs (small systems) against launched ones: the
same kernels in the same order, hence the same bits, whatever buffers, initial
guesses, limits and streams the caller brings."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
amg = pytest.importorskip("paper_1503_01287_amd")
from paper_1503_01287_amd import problems

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("krylov,precision", [("PCG", "FP64"), ("FCG", "FP64"), ("FCG", "MIXED")])
@pytest.mark.parametrize("problem,n", [("laplace", 3), ("elasticity", 6)])
def test_same_bits(problem, n, krylov, precision):
    sysm = getattr(problems, problem)(n)
    kw = dict(krylov=krylov, precision=precision, autotune=False)
    rec, eager = amg.AMGSolver(sysm, **kw), amg.AMGSolver(sysm, graph=False, **kw)
    rng = np.random.default_rng(n)
    side = torch.cuda.Stream()
    for k in range(6):
        b = torch.from_numpy(sysm.rhs if k == 0 else rng.standard_normal(sysm.dofs)).cuda()
        x0 = torch.zeros_like(b) if k < 2 else torch.from_numpy(rng.standard_normal(sysm.dofs)).cuda()
        torch.cuda.synchronize()
        got = []
        for s in (rec, eager):
            x = x0.clone()
            with torch.cuda.stream(side if k % 2 else torch.cuda.current_stream()):
                torch.cuda.current_stream().wait_stream(torch.cuda.default_stream())
                r = s.solve(b, x, tol=1e-10, maxit=3 if k == 5 else 200)
                torch.cuda.current_stream().synchronize()
            got.append((x, r.iters, r.status, r.relres))
        assert torch.equal(got[0][0], got[1][0]), k
        assert got[0][1:] == got[1][1:], k
        assert (got[0][1] == 3) == (k == 5)
