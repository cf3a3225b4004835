"""The counts of expansions behind fmm_far_evals and the algorithmic FLOP are those
the rows need: one where a root lies out of reach of its last one.  Expansions that
lanes get along with another's are not counted.  Against a count made here, root
by root, from the rows that come back: a root's reach from the stars around it, and a
new centre three quarters of the last reach ahead."""
import numpy as np
import pytest
import torch

from paper_2506_02121_amd import fields

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.as_tensor(np.array(a, copy=True), dtype=torch.float64).cuda()


def reach(z, stars, m):
    """14 moments, terms left out below 2e-17 of sum m |u|^2."""
    u2 = 1.0 / np.abs(z[:, None] - stars[None, :]) ** 2
    x = 0.95 * (2e-17 / 14 * u2.max(axis=1) / (m * u2 * u2).sum(axis=1)) ** (1.0 / 13)
    return np.minimum(x, 0.25) / np.sqrt(u2.max(axis=1))


def needed(rows, stars, m, centre):
    n = 0
    for d, end in ((-1, -1), (1, rows.shape[0])):
        c, r = rows[centre].copy(), np.full(rows.shape[1], -1.0)
        prev = rows[centre]
        for j in range(centre + d, end, d):
            z = rows[j]
            out = np.abs(z - c) > r
            v = z - prev
            a = np.abs(v)
            lead = np.where((r > 0) & (a > 0), 0.75 * r / np.maximum(a, 1e-300), 0.0)
            c = np.where(out, z + lead * v, c)
            r = np.where(out, reach(c, stars, m), r)
            again = np.abs(z - c) > r   # still too far: at its own place
            c = np.where(again, z, c)
            r = np.where(again, reach(c, stars, m), r)
            n += int(out.sum() + again.sum())
            prev = z
    return n


# all 2 n roots in one block, so that no sweep takes the multipole sums
@pytest.mark.parametrize("n,m_steps", [(4, 1200), (8, 2000)])
def test_only_what_a_root_needs_is_counted(n, m_steps):
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2506_02121_amd import mlcc
    print("[case]", n, m_steps, flush=True)
    f = fields.random_field(23, n, kappa_star=0.4, gamma=0.3, masses="salpeter")
    ctx = mlcc.Context(0)
    ctx.set_lenses(dev(f.x), dev(f.y), dev(f.m), f.kappa_s, f.gamma)
    re, im, _, s, _ = ctx.find_critical_curves(m_steps, n_subchains=1, star_sums="fmm")
    rows = re.cpu().numpy() + 1j * im.cpu().numpy()
    ctx.close()
    want = needed(rows, f.x + 1j * f.y, f.m, m_steps // 2)
    print("[tallies]", s["fmm_far_evals"], want, flush=True)
    # a row of a root left open is taken again, and centres start from predictions:
    # a tenth for both; fewer where another root's turn came first
    assert 0 < s["fmm_far_evals"] <= 1.1 * want
