"""The persistent launch's work groups: fronts of 1 to 8 blocks of 64 roots
are run whole by one work group, longer ones in tasks of four blocks through
the queue.  At the sizes where that choice and the last, partly filled task
change, both schedules run the same passes, so the results agree bit for bit."""
import numpy as np
import pytest
import torch

from paper_2506_02121_amd import fields

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mlcc():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2506_02121_amd import mlcc as m
    return m


def dev(a):
    return torch.as_tensor(np.array(a, copy=True), dtype=torch.float64).cuda()


def both(ctx, m_steps, **kw):
    out = []
    for sched in ("rounds", "persistent"):
        r = ctx.find_critical_curves(m_steps, caustics=True, schedule=sched, **kw)
        torch.cuda.synchronize()
        out.append(([t.cpu().numpy() for t in r[:5]], r[5]))
    (a, sa), (b, sb) = out
    for x, y in zip(a, b):
        assert np.array_equal(x.view(np.uint8), y.view(np.uint8))
    for k in ("root_updates", "root_updates_f32", "polish_updates", "rows_fallback"):
        assert sa[k] == sb[k], k


# 1 block; exactly one; two; 4; 5; 8; 9 blocks (queued: 4 + 4 + 1); 13 (4 x 3 + 1)
@pytest.mark.parametrize("n", [1, 32, 33, 128, 160, 256, 257, 400])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_front_lengths(mlcc, n, precision):
    print("[case]", n, precision, flush=True)
    ctx = mlcc.Context(0)
    f = fields.random_field(41, n, kappa_star=0.45, kappa_s=0.05, gamma=0.27, masses="salpeter")
    ctx.set_lenses(dev(f.x), dev(f.y), dev(f.m), f.kappa_s, f.gamma)
    both(ctx, 96, n_subchains=3, precision=precision)
    ctx.close()


@pytest.mark.parametrize("star_sums", ["direct", "fmm"])
def test_batch_of_unequal_lengths(mlcc, star_sums):
    """Owned and queued fronts side by side: the longest field decides the
    work group, and the short ones make one task each."""
    print("[case] batch", star_sums, flush=True)
    ctx = mlcc.Context(0)
    fs = [fields.random_field(50 + i, n, kappa_star=0.4, gamma=0.3, masses="salpeter")
          for i, n in enumerate([3, 33, 128, 129, 300])]
    off = np.concatenate([[0], np.cumsum([f.n for f in fs])])
    cat = [dev(np.concatenate([getattr(f, k) for f in fs])) for k in ("x", "y", "m")]
    ctx.set_lenses_batched(list(off), *cat, [f.kappa_s for f in fs], [f.gamma for f in fs])
    both(ctx, 64, n_subchains=2, precision="fp64", star_sums=star_sums)
    ctx.close()
