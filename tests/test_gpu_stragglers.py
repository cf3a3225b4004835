"""Blocks with at most 16 roots left, whose roots the whole wave takes one at a
time: star and root counts either side of the 256 records that are loaded four a
lane, with a last block of 2 to 8 roots, so that every sweep of it goes this way.
Rows against the oracle's, root by root."""
import numpy as np
import pytest
import torch

import oracle
from paper_2506_02121_amd import fields
from tests import parity

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.as_tensor(np.array(a, copy=True), dtype=torch.float64).cuda()


# 2 n roots: 2, 16, 130 .. 258 (one load group and 2 records), 514, 520 (two, and the rest);
# 257 and 260 stars: one group and 1 and 4 records
@pytest.mark.parametrize("n", [1, 8, 65, 128, 129, 256, 257, 260])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("masses", ["equal", "salpeter"])
def test_few_roots_of_a_block(n, masses, precision):
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2506_02121_amd import mlcc
    print("[case]", n, masses, precision, flush=True)
    m_steps = 24
    f = fields.random_field(17, n, kappa_star=0.4, kappa_s=0.05, gamma=0.3, masses=masses)
    ctx = mlcc.Context(0)
    ctx.set_lenses(dev(f.x), dev(f.y), dev(f.m), f.kappa_s, f.gamma)
    re, im = ctx.find_critical_curves(m_steps, n_subchains=1, precision=precision)[:2]
    rows = re.cpu().numpy() + 1j * im.cpu().numpy()
    ctx.close()
    ref, _, _ = oracle.critical_curves(f, m_steps, n_sub=1)
    slope = np.stack([oracle.eval_F(f, oracle.phase(j, m_steps), ref[j])[1]
                      for j in range(m_steps + 1)])
    _, ratio = parity.compare_row_sets(rows, ref, parity.root_bound(f, slope))
    assert ratio <= 1.0
