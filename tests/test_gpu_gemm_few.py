"""bf16 projections of few tiles (32 x 32 per block, a ring of 16 k-tiles): the epilogues that one call can ask for, at the edges of the tile, of the ring and of the rule."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N", [(1, 1), (31, 33), (65, 95), (512, 512), (513, 480), (33, 3072)])   # (513, 512) is past the rule's 256 tiles
@pytest.mark.parametrize("K", [64, 128, 192, 15 * 64, 16 * 64, 17 * 64, 18 * 64, 3072])
def test_few_tiles_match_fp64(M, N, K):
    import torch
    from paper_2601_12917_amd import binding as B
    gen = torch.Generator().manual_seed(M + N + K)
    A, W, b = (torch.randn(*s, generator=gen).mul(f).bfloat16() for s, f in (((M, K), 1.0), ((N, K), K ** -0.5), ((N,), 1.0)))
    old = torch.randn(M, N, generator=gen)
    x = A.double() @ W.double().T + b.double()
    # exact products, each of the K sums rounding to 2^-24 of what it holds, a random walk; |gelu'| <= 1.13, and gelu in fp32 to 2^-20
    walk = 4 * np.sqrt(K + 16) * 2.0 ** -24 * 1.13 * (A.double().abs() @ W.double().abs().T + b.double().abs() + 1.0) + 2.0 ** -20
    Ad, Wd, bd = A.cuda(), W.cuda(), b.cuda()
    for epi, want in ((0, x), (1, 0.5 * x * (1 + torch.erf(x / 2 ** 0.5))), (2, old.double() + x), (3, x)):
        out = old.cuda() if epi == 2 else torch.full((M, N), 7.0, device="cuda", dtype=torch.float32 if epi == 3 else torch.bfloat16)
        B.check(B.lib().zgr_debug_gemm(1, Ad.data_ptr(), Wd.data_ptr(), bd.data_ptr(), out.data_ptr(), epi, M, N, K, torch.cuda.current_stream().cuda_stream))
        torch.cuda.synchronize()
        store = 0.0 if epi in (2, 3) else 2.0 ** -8 * want.abs()   # half a unit in the last place of bf16
        assert torch.all((out.double().cpu() - want).abs() <= walk + store), epi
