"""The fused vector passes of a batch's conjugate gradients (update of x and r
with <r, r>, and of the search direction, step lengths in pinned host
memory): batches of one system, of systems below, just past and some chunks
past the 2,048 unknowns of a workgroup, and of more systems than a wavefront
has lanes, each solved twice with one solver object. The oracle is each
system's own solve; both stop at a relative residual of 1e-12, which leaves
the solutions within twice 1e-12 times the condition number (below KAPPA on
these meshes) of each other in the 2-norm."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_1503_01287_amd as amg  # noqa: E402

DEV = torch.device("cuda:0")
KAPPA = 1000.0  # 375 at n = 6, 146 at n = 3
SIZES = {"one": [3], "chunks": [1, 4, 5, 2, 6], "many": [1, 2, 2, 1, 3] * 14}


@pytest.mark.parametrize("krylov,precision", [("PCG", "FP64"), ("FCG", "MIXED")])
@pytest.mark.parametrize("sizes", list(SIZES))
def test_batch_cg_matches_own_solves(sizes, krylov, precision):
    ns = SIZES[sizes]
    meshes = {n: amg.problems.laplace(n) for n in set(ns)}
    systems = [meshes[n] for n in ns]
    bs = amg.BatchedSolver(systems, smoother="GS-1-1", krylov=krylov, precision=precision)
    rng = np.random.default_rng(17)
    for scale in (1.0, 1e6):
        b = [scale * (k + 1) * meshes[n].rhs + 1e-3 * scale * rng.standard_normal(meshes[n].dofs)
             for k, n in enumerate(ns)]
        x = torch.zeros(bs.n, dtype=torch.float64, device=DEV)
        res = bs.solve(torch.from_numpy(np.concatenate(b)).to(DEV), x, tol=1e-12, maxit=300)
        X = x.cpu().numpy()
        singles = {n: amg.AMGSolver(meshes[n], smoother="GS-1-1", krylov="PCG") for n in set(ns)}
        o = 0
        for k, n in enumerate(ns):
            assert res[k].converged, (k, n, res[k])
            x1 = torch.zeros(meshes[n].dofs, dtype=torch.float64, device=DEV)
            singles[n].solve(torch.from_numpy(b[k]).to(DEV), x1, tol=1e-12, maxit=300)
            x1 = x1.cpu().numpy()
            assert np.linalg.norm(X[o:o + x1.size] - x1) <= 2e-12 * KAPPA * np.linalg.norm(x1), (k, n, scale)
            o += x1.size
        for s in singles.values():
            s.close()
    bs.close()
