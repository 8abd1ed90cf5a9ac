"""Patterns that hold (i, j) and not (j, i): the greedy colouring looks at a
row's own entries, so i < j may share a colour, and a row that waited inside a
sweep for one of its own colour would wait for ever. Such levels run one launch
per colour, where row i reads x_j either before or after its update."""
import copy

import numpy as np
import pytest

torch = pytest.importorskip("torch")
amg = pytest.importorskip("paper_1503_01287_amd")
from paper_1503_01287_amd import problems

DEV = "cuda"
MAKE = {"laplace": problems.laplace, "elasticity": problems.elasticity}


def greedy(ptr, col):
    colour = np.full(len(ptr) - 1, -1)
    for i in range(len(colour)):
        taken = set(colour[col[ptr[i]:ptr[i + 1]]])
        colour[i] = next(c for c in range(len(colour)) if c not in taken)
    return colour


def insert(ptr, col, val, i, j, entry):
    """The arrays with the entry (i, j) added."""
    at = ptr[i] + np.searchsorted(col[ptr[i]:ptr[i + 1]], j)
    assert at == ptr[i + 1] or col[at] != j
    w = len(entry)
    ptr = ptr.copy()
    ptr[i + 1:] += 1
    return ptr, np.insert(col, at, j).astype(np.int32), np.insert(val.reshape(-1, w), at, entry, 0).reshape(-1).copy()


def uncoupled_pair(ptr, col):
    """i < j of one colour, as far apart as there are."""
    colour = greedy(ptr, col)
    i = 0
    j = np.flatnonzero(colour == colour[i])[-1]
    assert j > i and j not in col[ptr[i]:ptr[i + 1]] and i not in col[ptr[j]:ptr[j + 1]]
    return i, int(j)


def one_sided(sysm, scale):
    i, j = uncoupled_pair(sysm.A_rowptr, sysm.A_col)
    w = sysm.bs * sysm.bs
    diag = sysm.A_val.reshape(-1, w)[sysm.A_rowptr[i]:sysm.A_rowptr[i + 1]].reshape(-1, w)
    entry = scale * np.abs(diag).max() * (np.eye(3) + 0.5).ravel()[:w]
    out = copy.copy(sysm)
    out.A_rowptr, out.A_col, out.A_val = insert(sysm.A_rowptr, sysm.A_col, sysm.A_val, i, j, entry)
    return out, i, j


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def sweep(s, colour, b, x, forward, pair, late):
    """A sweep by colours; of the coupled pair, j's row before i's if late."""
    x, n, k = x.copy().reshape(-1, 3), len(colour), s.bs
    val = s.A_val.reshape(-1, k, k)
    for c in sorted(set(colour), reverse=not forward):
        rows = list(np.flatnonzero(colour == c))
        if late and pair[1] in rows:
            rows.remove(pair[1])
            rows.insert(0, pair[1])
        for i in rows:
            r, d = b.reshape(-1, 3)[i].copy(), None
            for q in range(s.A_rowptr[i], s.A_rowptr[i + 1]):
                e = val[q] if k == 3 else val[q, 0, 0] * np.eye(3)
                r -= e @ x[s.A_col[q]]
                if s.A_col[q] == i:
                    d = e
            x[i] += np.linalg.solve(d, r)
    return x.reshape(-1)


def test_the_pair_shares_a_colour():
    for make in MAKE.values():
        s, i, j = one_sided(make(3), 0.1)
        colour = greedy(s.A_rowptr, s.A_col)
        assert colour[i] == colour[j] and j in s.A_col[s.A_rowptr[i]:s.A_rowptr[i + 1]]


@pytest.mark.gpu
@pytest.mark.parametrize("problem", list(MAKE))
@pytest.mark.parametrize("n", [2, 4])
def test_one_sweep(problem, n):
    s, i, j = one_sided(MAKE[problem](n), 0.1)
    solver = amg.AMGSolver(s, autotune=False, fuse_coarse=False)
    colour = solver.level_colors(0)
    assert colour[i] == colour[j]
    rng = np.random.default_rng(n)
    b, x = rng.standard_normal(s.dofs), rng.standard_normal(s.dofs)
    for forward in (True, False):
        got = dev(x)
        solver.smooth(0, dev(b), got, forward)
        got = got.cpu().numpy()
        off = [np.abs(got - w).max() / np.abs(w).max()
               for w in (sweep(s, colour, b, x, forward, (i, j), late) for late in (False, True))]
        assert min(off) < 1e-11, off  # at most 14 dependent colours of 65 blocks, 1e-16 each


@pytest.mark.gpu
@pytest.mark.parametrize("problem", list(MAKE))
@pytest.mark.parametrize("precision", ["FP64", "FP32", "MIXED"])
def test_cycle_and_solve(problem, precision):
    """A coupling of 1e-7 of the diagonal changes a cycle by about as much
    (FP32 and BF16 operators: by their own rounding)."""
    s = MAKE[problem](5)
    t, _, _ = one_sided(s, 1e-7)
    kw = dict(smoother="GS-2-2", krylov="FCG", precision=precision)
    one, two = amg.AMGSolver(s, **kw), amg.AMGSolver(t, **kw)
    r = dev(np.random.default_rng(5).standard_normal(s.dofs))
    z, w = torch.zeros_like(r), torch.zeros_like(r)
    one.precondition(r, z)
    for _ in range(3):  # replays
        two.precondition(r, w)
        assert float((z - w).abs().max() / z.abs().max()) < 1e-4
    x = torch.zeros_like(r)
    assert two.solve(dev(t.rhs), x, tol=1e-6).converged


@pytest.mark.gpu
@pytest.mark.parametrize("precision", ["FP64", "MIXED"])
def test_batch(precision):
    a, b = problems.elasticity(4), problems.elasticity(6)
    c, _, _ = one_sided(b, 1e-7)
    kw = dict(smoother="GS-1-1", krylov="FCG", precision=precision)
    one, two = amg.BatchedSolver([a, b], **kw), amg.BatchedSolver([a, c], **kw)
    r = dev(np.random.default_rng(6).standard_normal(a.dofs + b.dofs))
    z, w = torch.zeros_like(r), torch.zeros_like(r)
    one.precondition(r, z)
    two.precondition(r, w)
    assert float((z - w).abs().max() / z.abs().max()) < 1e-4


@pytest.mark.gpu
@pytest.mark.parametrize("precision", ["FP64", "FP32"])
def test_schur_complement(precision):
    """C of a saddle point system one-sided: a Schur level's sweeps."""
    s = problems.mixed_elasticity(5)
    m, nodes = s.n_pres, s.nodes
    B, C = np.zeros((m, nodes), bool), np.zeros((m, m), bool)
    B[np.repeat(np.arange(m), np.diff(s.B_rowptr)), s.B_col] = True
    C[np.repeat(np.arange(m), np.diff(s.C_rowptr)), s.C_col] = True
    S = (B.astype(int) @ B.T.astype(int) > 0) | C
    ptr = np.concatenate([[0], np.cumsum(S.sum(1))])
    i, j = uncoupled_pair(ptr, np.nonzero(S)[1])
    t = copy.copy(s)
    t.C_rowptr, t.C_col, t.C_val = insert(s.C_rowptr, s.C_col, s.C_val, i, j, [1e-7 * np.abs(s.C_val).max()])
    kw = dict(smoother="BS-1-1", krylov="FGMRES", precision=precision)
    one, two = amg.AMGSolver(s, **kw), amg.AMGSolver(t, **kw)
    r = dev(np.random.default_rng(7).standard_normal(s.dofs))
    z, w = torch.zeros_like(r), torch.zeros_like(r)
    one.precondition(r, z)
    two.precondition(r, w)
    assert float((z - w).abs().max() / z.abs().max()) < 1e-4
