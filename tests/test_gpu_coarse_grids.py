"""Phase grids too coarse for expansions of the star field (below 256 steps in
FP64, 400 in the mixed form) take every warm row by passes alone: the work counts
are those of sums over all stars and roots, update by update.  From those step
counts on rows come from expansions, whose work is counted otherwise."""
import numpy as np
import pytest
import torch

from paper_2506_02121_amd import fields

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.as_tensor(np.array(a, copy=True), dtype=torch.float64).cuda()


@pytest.mark.parametrize("schedule", ["persistent", "rounds"])
@pytest.mark.parametrize("precision,m_steps,expands",
                         [("fp64", 2, False), ("fp64", 96, False), ("fp64", 254, False),
                          ("fp64", 256, True), ("fp64_r32", 254, False), ("fp64_r32", 256, True),
                          ("mixed", 96, False), ("mixed", 398, False), ("mixed", 400, True)])
def test_rows_by_passes_alone(precision, m_steps, expands, schedule):
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2506_02121_amd import mlcc
    print("[case]", precision, m_steps, schedule, flush=True)
    n = 150
    f = fields.random_field(8, n, kappa_star=0.5, gamma=0.3, masses="salpeter")
    ctx = mlcc.Context(0)
    ctx.set_lenses(dev(f.x), dev(f.y), dev(f.m), f.kappa_s, f.gamma)
    s = ctx.find_critical_curves(m_steps, precision=precision, schedule=schedule)[3]
    ctx.close()
    star, root = 29.0 * n, 10.0 * (2 * n - 1)
    if precision == "mixed":
        got, want = s["algorithmic_flop_polish"], star * s["polish_updates"]
    else:
        got = s["algorithmic_flop"] + s["algorithmic_flop_sweep_roots"]
        want = (star + root) * s["root_updates"]
    assert (got == want) == (not expands)
