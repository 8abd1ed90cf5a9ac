"""Vanka sweeps in one launch where a patch has more unknowns than the columns
that a lane loads before it waits (416), and a row more entries than are ranked
by their writers (1,024)."""
import copy

import numpy as np
import pytest

torch = pytest.importorskip("torch")
amg = pytest.importorskip("paper_1503_01287_amd")
from paper_1503_01287_amd import problems

pytestmark = pytest.mark.gpu


def grow(ptr, col, val, i, add):
    """Row i with the entries `add` {column: values} as well."""
    w = len(val) // len(col)
    row = {int(col[k]): val[k * w:(k + 1) * w] for k in range(ptr[i], ptr[i + 1])}
    row = {**add, **row}
    cols = sorted(row)
    new = np.concatenate([row[c] for c in cols])
    out = ptr.copy()
    out[i + 1:] += len(cols) - (ptr[i + 1] - ptr[i])
    return (out, np.concatenate([col[:ptr[i]], cols, col[ptr[i + 1]:]]).astype(np.int32),
            np.concatenate([val[:w * ptr[i]], new, val[w * ptr[i + 1]:]]))


def system(patch, row):
    """Mixed elasticity 5^3 with a pressure coupled to `patch` more nodes and a
    node coupled to `row` others."""
    s = copy.copy(problems.mixed_elasticity(5, nu=0.4))
    rng = np.random.default_rng(patch + row)
    scale = 1e-3 * np.abs(s.B_val).max()
    extra = rng.choice(s.nodes, patch, replace=False)
    s.B_rowptr, s.B_col, s.B_val = grow(s.B_rowptr, s.B_col, s.B_val, 100,
                                        {int(j): scale * rng.standard_normal(3) for j in extra})
    u, scale = 700, 1e-4 * np.abs(s.A_val).max()
    others = [int(j) for j in rng.choice(s.nodes, row, replace=False) if j != u]
    blocks = {j: scale * rng.standard_normal(9) for j in others}
    s.A_rowptr, s.A_col, s.A_val = grow(s.A_rowptr, s.A_col, s.A_val, u, blocks)
    for j in others:
        s.A_rowptr, s.A_col, s.A_val = grow(s.A_rowptr, s.A_col, s.A_val, j,
                                            {u: blocks[j].reshape(3, 3).T.reshape(-1)})
    return s


@pytest.mark.parametrize("patch,row", [(90, 0), (260, 0), (0, 1150), (260, 1150)])
def test_one_launch_equals_launch_per_colour(patch, row):
    s = system(patch, row)
    if patch == 260:
        assert 3 * (s.B_rowptr[101] - s.B_rowptr[100]) > 800
    if row:
        assert s.A_rowptr[701] - s.A_rowptr[700] > 1024
    one, per = (amg.AMGSolver(s, smoother="Vanka-1-1", krylov="FGMRES", autotune=False) for _ in range(2))
    per.set_launch_shape(0, "vanka_apply", 8)
    rng = np.random.default_rng(5)
    b, x = (torch.from_numpy(rng.standard_normal(s.dofs)).cuda() for _ in range(2))
    y = x.clone()
    for k in range(4):  # the buffers are turned over after every sweep
        one.smooth(0, b, x)
        per.smooth(0, b, y)
        # sums of at most 1,200 products in another order, each patch's error
        # carried through the later ones: as for the oracle, 1e-10
        assert float((x - y).abs().max() / y.abs().max()) < 1e-10, k
