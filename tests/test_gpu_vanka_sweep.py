"""Vanka sweeps with all colours in one launch against a launch per colour."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
amg = pytest.importorskip("paper_1503_01287_amd")
from paper_1503_01287_amd import problems

pytestmark = pytest.mark.gpu

SYSTEMS = {  # rows of 1 to 200 entries, patches of 13 to 400 unknowns
    "mixed2": lambda: problems.mixed_elasticity(2, nu=0.3),
    "mixed3": lambda: problems.mixed_elasticity(3),
    "mixed6": lambda: problems.mixed_elasticity(6, nu=0.4),
    "mixed9": lambda: problems.mixed_elasticity(9),
    "cavity5": lambda: problems.stokes_cavity(5, 1.1),
}


def pair(name):
    s = SYSTEMS[name]()
    one, per = (amg.AMGSolver(s, smoother="Vanka-1-1", krylov="FGMRES", autotune=False) for _ in range(2))
    for l in range(per.num_levels - 1):
        per.set_launch_shape(l, "vanka_apply", 8)
    return s, one, per


@pytest.mark.parametrize("name", list(SYSTEMS))
def test_one_launch_equals_launch_per_colour(name):
    s, one, per = pair(name)
    rng = np.random.default_rng(5)
    for l in range(one.num_levels - 1):
        n = one.level_dofs(l)
        b = torch.from_numpy(rng.standard_normal(n)).cuda()
        x = torch.from_numpy(rng.standard_normal(n)).cuda()
        y = x.clone()
        for k in range(5):  # the buffers are turned over after every sweep
            one.smooth(l, b, x)
            per.smooth(l, b, y)
            # sums of at most 400 products in another order, each patch's
            # error carried through the later ones: as for the oracle, 1e-10
            assert float((x - y).abs().max() / y.abs().max()) < 1e-10, (l, k)
    r = torch.from_numpy(rng.standard_normal(s.dofs)).cuda()
    z, w = torch.zeros_like(r), torch.zeros_like(r)
    for k in range(4):  # the later ones replay a recorded graph
        one.precondition(r, z)
        per.precondition(r, w)
        torch.cuda.synchronize()
        assert float((z - w).abs().max() / w.abs().max()) < 1e-9, k
        r = r.roll(1) + 1.0


@pytest.mark.parametrize("bits", [0x7FF8000000000000, 0x7FF0000000000000, 0x7FFDEAD0BEEF0001])
@pytest.mark.parametrize("where", ["b", "x"])
def test_nan_and_infinity_end(bits, where):
    """Also a NaN with the payload of a value that is not there yet: the
    sweep ends, spreads it, and leaves the next sweep right."""
    _, one, per = pair("mixed3")
    n = one.level_dofs(0)
    rng = np.random.default_rng(6)
    b, x = rng.standard_normal(n), rng.standard_normal(n)
    (b if where == "b" else x).view(np.uint64)[n // 2] = bits
    b, x = torch.from_numpy(b).cuda(), torch.from_numpy(x).cuda()
    y = x.clone()
    one.smooth(0, b, x)
    per.smooth(0, b, y)
    assert torch.equal(torch.isfinite(x), torch.isfinite(y)) and not torch.isfinite(x).all()
    b, x = (torch.from_numpy(rng.standard_normal(n)).cuda() for _ in range(2))
    y = x.clone()
    one.smooth(0, b, x)
    per.smooth(0, b, y)
    assert float((x - y).abs().max() / y.abs().max()) < 1e-10
