"""Schur complement sweeps in one launch against a launch per colour. A zero
entry (i, j) of C without (j, i), i and j of one colour, changes no value but
keeps the finest Schur level from the one launch."""
import copy

import numpy as np
import pytest

torch = pytest.importorskip("torch")
amg = pytest.importorskip("paper_1503_01287_amd")
from paper_1503_01287_amd import problems

pytestmark = pytest.mark.gpu


def greedy(ptr, col):
    colour = np.full(len(ptr) - 1, -1)
    for i in range(len(colour)):
        taken = set(colour[col[ptr[i]:ptr[i + 1]]])
        colour[i] = next(c for c in range(len(colour)) if c not in taken)
    return colour


def with_a_zero(s):
    m = s.n_pres
    B, C = np.zeros((m, s.nodes), np.float32), np.zeros((m, m), bool)
    B[np.repeat(np.arange(m), np.diff(s.B_rowptr)), s.B_col] = 1
    C[np.repeat(np.arange(m), np.diff(s.C_rowptr)), s.C_col] = True
    S = (B @ B.T > 0) | C
    colour = greedy(np.concatenate([[0], np.cumsum(S.sum(1))]), np.nonzero(S)[1])
    i, j = next((a, b) for a in range(m) for b in range(m - 1, a, -1) if colour[a] == colour[b])
    assert not S[i, j]
    at = s.C_rowptr[i] + np.searchsorted(s.C_col[s.C_rowptr[i]:s.C_rowptr[i + 1]], j)
    t = copy.copy(s)
    t.C_rowptr = s.C_rowptr.copy()
    t.C_rowptr[i + 1:] += 1
    t.C_col, t.C_val = np.insert(s.C_col, at, j).astype(np.int32), np.insert(s.C_val, at, 0.0)
    return t


@pytest.mark.parametrize("precision", ["FP64", "FP32"])
@pytest.mark.parametrize("smoother", ["BS-1-1", "BS-2-1"])
@pytest.mark.parametrize("n", [4, 6, 9])  # 125, 343 and 1,000 rows, the last tiles of a colour partly filled
def test_same_cycle(n, smoother, precision):
    s = problems.mixed_elasticity(n, nu=0.45)
    kw = dict(smoother=smoother, krylov="FGMRES", precision=precision, autotune=False, fuse_coarse=False)
    one, per = amg.AMGSolver(s, **kw), amg.AMGSolver(with_a_zero(s), **kw)
    r = torch.from_numpy(np.random.default_rng(n).standard_normal(s.dofs)).cuda()
    z, w = torch.zeros_like(r), torch.zeros_like(r)
    for k in range(3):
        one.precondition(r, z)
        per.precondition(r, w)
        # the same products in another order: rows of at most some 130 terms
        # over 30 dependent colours, 1e-16 (6e-8) each
        assert float((z - w).abs().max() / w.abs().max()) < (1e-11 if precision == "FP64" else 1e-4), k
        r = r.roll(1)
