"""The finest level's operator in tiles (large scalar systems) against SciPy
and against the row kernels."""
import numpy as np
import pytest
import scipy.sparse as sp

torch = pytest.importorskip("torch")
amg = pytest.importorskip("paper_1503_01287_amd")
from paper_1503_01287_amd import problems

pytestmark = pytest.mark.gpu


def matrix(s):
    return sp.csr_matrix((s.A_val, s.A_col, s.A_rowptr), shape=(s.nodes,) * 2)


def circulant(n, half):
    """SPD rows of 2 half + 1 entries at distances without locality: 256 rows
    read far more nodes than a tile may."""
    off = np.unique(np.random.default_rng(0).integers(1, n // 2, size=half))
    cols = (np.arange(n)[:, None] + np.concatenate([[0], off, n - off])[None, :]) % n
    vals = np.full(cols.shape, -1.0)
    vals[:, 0] = 2 * off.size + 1
    order = np.argsort(cols, axis=1)
    rowptr = np.arange(n + 1, dtype=np.int32) * cols.shape[1]
    return problems.LinearSystem("circulant", 0, n, 0, 0, 1, rowptr,
                                 np.take_along_axis(cols, order, 1).astype(np.int32).ravel(),
                                 np.take_along_axis(vals, order, 1).ravel(), np.ones(3 * n), np.zeros((n, 3)))


@pytest.fixture(scope="module")
def cube():
    return problems.laplace(24)  # 117649 rows: 459 tiles and 145 rows


def solve(s, b):
    x = torch.zeros_like(b)
    res = s.solve(b, x, tol=1e-10)
    assert res.status == 0
    return x, res.iters


@pytest.mark.parametrize("precision,krylov", [("FP64", "PCG"), ("FP32", "FCG"), ("MIXED", "FCG")])
@pytest.mark.parametrize("smoother", ["JA-1-1-0.5", "JA-0-2-0.5", "GS-1-1"])
def test_tiles_equal_rows(cube, smoother, precision, krylov):
    kw = dict(smoother=smoother, krylov=krylov, precision=precision, autotune=False)
    tiles, rows = amg.AMGSolver(cube, **kw), amg.AMGSolver(cube, **kw)
    rows.set_launch_shape(0, "natural", 8)
    if precision != "FP64":
        rows.set_launch_shape(0, "natural_rp", 8)
    rng = np.random.default_rng(1)
    x = rng.standard_normal((cube.nodes, 3))
    A = matrix(cube)
    y = torch.zeros(cube.dofs, dtype=torch.float64, device="cuda")
    tiles.apply(0, torch.from_numpy(x.ravel()).cuda(), y)
    # a row's sum of at most 65 products in any order, twice
    bound = 2 * 66 * 2.0 ** -53 * (abs(A) @ np.abs(x)).ravel()
    assert (np.abs(y.cpu().numpy() - (A @ x).ravel()) <= bound).all()
    # each pass sums in another order than the rows'; the cycle is a
    # contraction, so one application stays within a few hundred roundings
    r = torch.from_numpy(rng.standard_normal(cube.dofs)).cuda()
    z, w = torch.zeros_like(r), torch.zeros_like(r)
    for _ in range(3):  # the later ones replay a recorded graph
        tiles.precondition(r, z)
    rows.precondition(r, w)
    assert float((z - w).norm() / w.norm()) < 512 * (2.0 ** -53 if precision == "FP64" else 2.0 ** -24)
    (u, iu), (v, iv) = solve(tiles, r), solve(rows, r)
    assert abs(iu - iv) <= 1
    assert float((u - v).norm() / v.norm()) < 1e-8


def test_infinities_stay_where_they_are_read(cube):
    s = amg.AMGSolver(cube, smoother="JA-1-1-0.5", autotune=False)
    A = matrix(cube)
    A.eliminate_zeros()
    x = np.ones((cube.nodes, 3))
    x[7, 1] = np.inf
    x[cube.nodes - 3, 2] = np.nan
    y = torch.zeros(cube.dofs, dtype=torch.float64, device="cuda")
    s.apply(0, torch.from_numpy(x.ravel()).cuda(), y)
    bad = np.zeros((cube.nodes, 3), dtype=bool)
    bad[A.tocsc()[:, 7].indices, 1] = True
    bad[A.tocsc()[:, cube.nodes - 3].indices, 2] = True
    assert (~np.isfinite(y.cpu().numpy().reshape(-1, 3)) == bad).all()


def test_rows_without_locality_keep_the_row_kernels():
    n = 110002
    c = circulant(n, 20)
    s = amg.AMGSolver(c, smoother="JA-1-1-0.5", krylov="FCG", precision="MIXED", autotune=False)
    x = np.random.default_rng(2).standard_normal((n, 3))
    y = torch.zeros(3 * n, dtype=torch.float64, device="cuda")
    s.apply(0, torch.from_numpy(x.ravel()).cuda(), y)
    A = matrix(c)
    assert (np.abs(y.cpu().numpy() - (A @ x).ravel()) <= 2 * 42 * 2.0 ** -53 * (abs(A) @ np.abs(x)).ravel()).all()
    solve(s, torch.from_numpy(x.ravel()).cuda())
