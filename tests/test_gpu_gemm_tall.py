"""The projection kernel for more than 128 activation rows at the edges of its tiles: 192, 256 and 320 rows
of X and 192 or 256 rows of W per workgroup, remainders of one row, several row blocks in one launch, one
to three 64-column stages, splits that end early."""
import pytest
import torch

from paper_2410_20488_amd import binding

pytestmark = pytest.mark.gpu

ROWS = [129, 192, 193, 256, 257, 320, 321, 577, 1024]
SHAPES = [(4, 64), (192, 128), (196, 192), (256, 64), (260, 320), (1000, 704), (4096, 1088)]


@pytest.mark.parametrize("n,K", SHAPES)
@pytest.mark.parametrize("rows", ROWS)
def test_tall_projection_at_tile_edges(rows, n, K):
    g = torch.Generator().manual_seed(rows * 7919 + n * 31 + K)
    x = torch.randn(rows, K, generator=g)
    w = torch.randn(n, K, generator=g).to(torch.bfloat16)
    y = binding.debug_gemm(x.cuda(), w.cuda(), kind=1).cpu().double()
    xd, wd = x.double(), w.double()
    # two bf16 planes hold x to 2^-18 of its size; 2K products are added in fp32 (2^-24 each at worst)
    bound = (2.0 ** -18 + 2 * K * 2.0 ** -24) * (xd.abs() @ wd.abs().T) + 1e-30
    assert bool(((y - xd @ wd.T).abs() <= bound).all())


def test_rows_of_a_tall_projection_do_not_depend_on_their_block():
    """Every row is computed by the same sums wherever its row block lies."""
    g = torch.Generator().manual_seed(5)
    row = torch.randn(1, 640, generator=g)
    w = torch.randn(516, 640, generator=g).to(torch.bfloat16).cuda()
    y = binding.debug_gemm(row.repeat(1024, 1).cuda(), w, kind=1)
    assert torch.equal(y, y[:1].expand_as(y))
