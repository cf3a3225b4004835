"""Every row of a coarse phase grid holds 2N distinct roots, the ones the oracle
finds.  A chain's extrapolation over a large phase step can land in the basin of
a neighbour's zero, so two columns can end at one root unless something keeps
them apart.  The fields below, among 600 of each size with seeds 0 .. 599, are
those where rows solved root by root had a root twice and another missing."""
import numpy as np
import pytest
import torch

import oracle
from paper_2506_02121_amd import fields
from tests import parity

pytestmark = pytest.mark.gpu

SEEDS = [(10, 8, (566,)),
         (40, 8, (76, 221, 582)), (40, 12, (313, 320)), (40, 20, (316,)),
         (150, 8, (6, 29, 89, 101, 103, 210, 289, 408, 420, 433, 490, 495, 513, 540, 564, 576)),
         (150, 12, (31, 45, 97, 331, 365, 383, 433)), (150, 16, (6, 36, 98, 159, 439)),
         (150, 20, (105,))]


@pytest.fixture(scope="module")
def mlcc():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2506_02121_amd import mlcc as m
    return m


def dev(a):
    return torch.as_tensor(np.array(a, copy=True), dtype=torch.float64).cuda()


@pytest.mark.parametrize("precision", ["fp64", "fp64_r32", "mixed"])
@pytest.mark.parametrize("schedule", ["persistent", "rounds"])
@pytest.mark.parametrize("n,m_steps,seeds", SEEDS)
def test_rows_hold_each_root_once(mlcc, n, m_steps, seeds, schedule, precision):
    print("[case]", n, m_steps, schedule, precision, flush=True)
    fs = [fields.random_field(s, n, kappa_star=0.7, kappa_s=0.1, gamma=0.1, masses="equal")
          for s in seeds]
    off = np.concatenate([[0], np.cumsum([f.n for f in fs])])
    cat = [dev(np.concatenate([getattr(f, k) for f in fs])) for k in ("x", "y", "m")]
    ctx = mlcc.Context(0)
    ctx.set_lenses_batched(list(off), *cat, [f.kappa_s for f in fs], [f.gamma for f in fs])
    re, im, cn, _, _ = ctx.find_critical_curves(m_steps, n_subchains=1, schedule=schedule,
                                                precision=precision)
    z = re.cpu().numpy() + 1j * im.cpu().numpy()
    blocks = ctx.field_blocks(m_steps)
    ctx.close()
    for f, (o, _, n_r) in zip(fs, blocks):
        rows = z[o:o + (m_steps + 1) * n_r].reshape(m_steps + 1, n_r)
        ref, _, _ = oracle.critical_curves(f, m_steps, n_sub=1)
        slope = np.stack([oracle.eval_F(f, oracle.phase(j, m_steps), ref[j])[1]
                          for j in range(m_steps + 1)])
        # pairs every root of a row with one of the oracle's, or fails
        _, ratio = parity.compare_row_sets(rows, ref, parity.root_bound(f, slope))
        assert ratio <= 1.0


@pytest.mark.parametrize("schedule", ["persistent", "rounds"])
@pytest.mark.parametrize("precision", ["fp64", "fp64_r32"])
def test_rows_whose_identities_fail(mlcc, schedule, precision):
    """Cutoffs of 1e-3 leave some roots of passes that far from their zeros: rows
    that hold them beside roots from expansions fail their identities, and all their
    roots take Aberth steps; the rows after them start anew."""
    print("[case]", schedule, precision, flush=True)
    m_steps, tol = 600, 1e-3
    f = fields.random_field(3, 300, kappa_star=0.45, kappa_s=0.0, gamma=0.3, masses="salpeter")
    ctx = mlcc.Context(0)
    ctx.set_lenses(dev(f.x), dev(f.y), dev(f.m), f.kappa_s, f.gamma)
    re, im, _, s, _ = ctx.find_critical_curves(m_steps, schedule=schedule, precision=precision,
                                               tol_step=tol, tol_inv_mu=tol)
    fine = ctx.find_critical_curves(m_steps, predictor=0)
    rows = re.cpu().numpy() + 1j * im.cpu().numpy()
    ref = fine[0].cpu().numpy() + 1j * fine[1].cpu().numpy()
    ctx.close()
    assert s["rows_fallback"] > 0
    slope = np.stack([oracle.eval_F(f, oracle.phase(j, m_steps), ref[j])[1]
                      for j in range(m_steps + 1)])
    _, ratio = parity.compare_row_sets(rows, ref, parity.root_bound(f, slope, tol))
    assert ratio <= 1.0
