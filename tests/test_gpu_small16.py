"""fp32 products of so few 32 x 32 tiles that 16 x 16 ones are taken, against 64 bits; both sides of the line."""
import pytest
import torch

import paper_2509_15148_amd as A
from util import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K", [(1, 1, 4), (1, 16, 8), (16, 16, 16), (17, 15, 20), (15, 33, 60), (33, 17, 64), (16, 48, 68), (320, 128, 512), (5, 130, 516),
                                   (40, 40, 1028), (100, 64, 2052), (31, 100, 4096),
                                   (128, 1024, 1024), (129, 1024, 1024), (128, 1024, 1028), (64, 1280, 1028), (65, 1280, 1028),
                                   (256, 256, 128), (256, 257, 128), (257, 256, 1024), (200, 512, 32), (200, 512, 36), (200, 512, 132), (200, 512, 800), (200, 512, 804)])
def test_products_in_tiles_of_16(M, N, K):
    """Edges of the tiles, fewer steps than wavefronts, partly filled steps and batches of steps, the most tiles for short and for long K, both sides of the lines in K."""
    announce("tiles of 16", M, N, K)
    assert A.atts_gemm_routes(torch.float32, M, N, K)[0].kernel == A.KERNEL_SMALL
    g = torch.Generator().manual_seed(M + N + K)
    a, w = torch.randn(M, K, generator=g), torch.randn(N, K, generator=g)
    room = torch.full((M + 1, N), 7.0, device="cuda")                  # a row behind the output stays as it is
    A.atts_gemm_nt(a.cuda(), w.cuda(), room[:M])
    torch.cuda.synchronize()
    ref = a.double() @ w.double().t()
    bound = 2.0 ** -24 * (K ** 0.5 + 8) * 2 * (a.double().abs() @ w.double().abs().t())     # fp32 sums of K products, any order
    assert bool(((room[:M].cpu().double() - ref).abs() <= bound).all()) and bool((room[M] == 7.0).all())
