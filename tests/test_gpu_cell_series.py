"""The two kernels that form the cells' series give the same coefficients to the
last bit, so a field's columns are numbered alike whichever of them its size and
company call for.  A few fields alone take a work group a cell, forty of them in one
call a lane a cell; an FP64 cold start and the sweeps after it follow every bit of
the series, and no other part of these calls differs between the two."""
import numpy as np
import pytest
import torch

from paper_2506_02121_amd import fields

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.as_tensor(np.array(a, copy=True), dtype=torch.float64).cuda()


# order 0 (48: rows of 56), 8 and 15 (16), 24 and 31 (32), 39 (40), 63 (64); 32 stars and
# 64 fill their tiles, 101 and 129 leave remainders
@pytest.mark.parametrize("order", [0, 8, 15, 24, 31, 39, 63])
@pytest.mark.parametrize("masses", ["equal", "salpeter"])
@pytest.mark.parametrize("n", [32, 64, 101, 129])
def test_rows_alone_and_among_many(n, masses, order):
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2506_02121_amd import mlcc
    print("[case]", n, masses, order, flush=True)
    f = fields.random_field(29, n, kappa_star=0.4, gamma=0.3, masses=masses)
    ctx = mlcc.Context(0)
    out = []
    for copies in (1, 40):
        ctx.set_lenses_batched([n * i for i in range(copies + 1)],
                               *(dev(np.tile(getattr(f, k), copies)) for k in ("x", "y", "m")),
                               [f.kappa_s] * copies, [f.gamma] * copies)
        # cleared, as a series of low order may leave rows unsolved
        res = tuple(torch.zeros(17 * 2 * n * copies, dtype=torch.float64, device="cuda")
                    for _ in range(2))
        r = ctx.find_critical_curves(16, n_subchains=2, star_sums="fmm", fmm_order=order,
                                     chain_next=False, raise_on_error=False, out=res)
        out.append((r[0].cpu().numpy().reshape(copies, -1),
                    r[1].cpu().numpy().reshape(copies, -1), r[4]))
    ctx.close()
    (ar, ai, ac), (br, bi, bc) = out
    assert ac == bc
    for i in range(br.shape[0]):
        assert np.array_equal(ar[0].view(np.int64), br[i].view(np.int64))
        assert np.array_equal(ai[0].view(np.int64), bi[i].view(np.int64))
