"""Flexible GMRES around an FP32 cycle whose right-hand side the
orthogonalisation writes: a fixed number of steps, restarts among them, with
the recorded cycle and without, by one solver object after a foreign
application, and in a batch, against the method written out with plain
vectors around the same solver's operator and preconditioner. The bound is
the FP32 cycle's own, 2e-4, for each of the steps."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_1503_01287_amd as amg  # noqa: E402

DEV = torch.device("cuda:0")


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).to(DEV)


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


def fgmres(A, M, b, m, steps):
    """`steps` steps of FGMRES(m) from zero."""
    x = np.zeros_like(b)
    while steps:
        r = b - A(x)
        V, Z, H = [r / np.linalg.norm(r)], [], np.zeros((m + 1, m))
        for j in range(min(m, steps)):
            Z.append(M(V[j]))
            w = A(Z[j])
            for _ in range(2):
                for i in range(j + 1):
                    c = V[i] @ w
                    H[i, j] += c
                    w = w - c * V[i]
            H[j + 1, j] = np.linalg.norm(w)
            V.append(w / H[j + 1, j])
            steps -= 1
        k = len(Z)
        e = np.zeros(k + 1)
        e[0] = np.linalg.norm(r)
        x = x + np.stack(Z, 1) @ np.linalg.lstsq(H[:k + 1, :k], e, rcond=None)[0]
    return x


@pytest.mark.parametrize("graph", [True, False])
@pytest.mark.parametrize("restart,steps", [(100, 1), (100, 6), (3, 5), (2, 4)])
def test_fgmres_steps(restart, steps, graph):
    s = amg.problems.mixed_elasticity(4, nu=0.3)
    sv = amg.AMGSolver(s, smoother="BS-1-1", krylov="FGMRES", precision="FP32", restart=restart, graph=graph)

    def op(f):
        def g(v):
            y = torch.zeros(s.dofs, dtype=torch.float64, device=DEV)
            f(dev(v), y)
            return host(y)
        return g

    ref = fgmres(op(lambda v, y: sv.apply(0, v, y)), op(sv.precondition), s.rhs, restart, steps)
    bound = 2e-4 * steps * np.linalg.norm(ref)
    batch = amg.BatchedSolver([s], smoother="BS-1-1", precision="FP32", restart=restart, graph=graph)
    for solver in (sv, batch, sv):
        x = torch.zeros(s.dofs, dtype=torch.float64, device=DEV)
        solver.solve(dev(s.rhs), x, tol=1e-300, maxit=steps)
        assert np.linalg.norm(host(x) - ref) <= bound, type(solver)
        sv.precondition(dev(np.ones(s.dofs)), x)
    batch.close()
    sv.close()
