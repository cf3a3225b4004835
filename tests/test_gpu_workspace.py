"""Device memory that a context takes for a mixed call beyond that of an FP64
call of the same field and pieces: partial row sums, 64 bytes for every block of 64
roots, and an error estimate a root.  It does not grow with the rows a block of
roots may be ahead of the others."""
import pytest
import torch

from paper_2506_02121_amd import fields

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("star_sums", ["direct", "fmm"])
def test_mixed_workspace(star_sums):
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2506_02121_amd import mlcc
    # 80 fronts of 129 blocks; 11 MiB by the sizes above, and what buffers round up to
    n, m_steps, n_sub = 4099, 160, 40
    f = fields.random_field(3, n, kappa_star=0.5, gamma=0.3, masses="salpeter")
    x, y, m = (torch.as_tensor(a, dtype=torch.float64).cuda() for a in (f.x, f.y, f.m))
    ctx = mlcc.Context(0)
    ctx.set_lenses(x, y, m, f.kappa_s, f.gamma)
    out = tuple(torch.empty((m_steps + 1, 2 * n), dtype=torch.float64, device="cuda")
                for _ in range(2))
    free = {}
    for precision in ("fp64", "mixed"):
        print("[case]", star_sums, precision, flush=True)
        ctx.find_critical_curves(m_steps, n_subchains=n_sub, chain_next=False, out=out,
                                 precision=precision, star_sums=star_sums)
        torch.cuda.synchronize()
        free[precision] = torch.cuda.mem_get_info()[0]
    ctx.close()
    assert free["fp64"] - free["mixed"] < 64 << 20
