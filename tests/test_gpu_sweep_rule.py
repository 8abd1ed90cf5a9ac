"""A level on either side of the line from which its sweeps take a launch per
colour: banded operators of two colours, so that few rows hold many entries."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
amg = pytest.importorskip("paper_1503_01287_amd")
from paper_1503_01287_amd.problems import LinearSystem

pytestmark = pytest.mark.gpu


def two_colours(m, reach=30):
    """Node i is coupled with the nodes i +- 1, 3, ..., 2 reach - 1."""
    offsets = np.concatenate([-np.arange(1, 2 * reach, 2)[::-1], [0], np.arange(1, 2 * reach, 2)])
    col = np.arange(m)[:, None] + offsets
    inside = (col >= 0) & (col < m)
    val = np.where(offsets == 0, 2.0, -1.0 / (4.0 * reach)) * np.ones((m, 1))
    ptr = np.concatenate([[0], np.cumsum(inside.sum(1))]).astype(np.int32)
    return LinearSystem("banded", 0, m, 0, 0, 1, ptr, col[inside].astype(np.int32), val[inside].copy(),
                        np.ones(3 * m), np.zeros((m, 3)))


@pytest.mark.parametrize("precision", ["FP64", "FP32", "MIXED"])
@pytest.mark.parametrize("smoother", ["GS-1-1", "GS-2-1", "GS-0-1"])
@pytest.mark.parametrize("m,launches", [(18000, 1), (21000, 2)])  # 540,000 and 630,000 entries a colour
def test_both_sides(m, launches, smoother, precision):
    s = two_colours(m)
    kw = dict(smoother=smoother, krylov="FCG", precision=precision)
    one, per = amg.AMGSolver(s, **kw), amg.AMGSolver(s, autotune=False, **kw)
    assert one.level_info(0).n_colors == 2
    for l in range(per.num_levels - 1):
        per.set_launch_shape(l, "sweep", 64)
        if precision != "FP64":
            per.set_launch_shape(l, "sweep_rp", 64)
    r = torch.from_numpy(np.random.default_rng(m).standard_normal(s.dofs)).cuda()
    z, w = torch.zeros_like(r), torch.zeros_like(r)
    per.precondition(r, w)
    for _ in range(3):  # replays
        one.precondition(r, z)
        # rows of 61 terms in another order: 1e-16 (6e-8) of them each
        assert float((z - w).abs().max() / w.abs().max()) < (1e-12 if precision == "FP64" else 1e-5)
    one.profile(1)
    one.precondition(r, z)
    torch.cuda.synchronize()
    sweeps = sum(int(v) for v in smoother.split("-")[1:])
    assert one.profile_read("gs.L0")["launches"] == launches * sweeps
    one.profile(0)
    x = torch.zeros_like(r)
    assert one.solve(r, x, tol=1e-6).converged
