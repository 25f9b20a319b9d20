"""fp32 products taken on the bf16 matrix instructions (an fp32 number as three bf16 numbers): both tile forms of the projections at
the edges of their tiles, k-tiles and dispatch rules, against fp64, and operands that are infinite, NaN or next to the largest number, which
have to give what fp32 products give."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

#          M     N     K
PRIVATE = [(767, 705, 192), (1024, 1024, 192), (320, 900, 640), (65, 4600, 672), (777, 770, 768), (1281, 1279, 640), (64, 4608, 3104)]      # 64 x 64 tiles, sums shared by four waves
SHARED = [(2048, 2048, 256), (1921, 2047, 288), (2048, 4096, 32), (129, 32769, 64), (4000, 2049, 96)]      # 128 x 128 tiles


@pytest.mark.parametrize("M,N,K", PRIVATE + SHARED)
@pytest.mark.parametrize("epi", [1, 2, 3], ids=["gelu", "add", "fp32"])
def test_projection_matches_fp64(M, N, K, epi):
    import torch
    from paper_2601_12917_amd import binding as B
    gen = torch.Generator().manual_seed(M + N + K + epi)
    A, W, b, old = (torch.randn(*s, generator=gen) * f for s, f in (((M, K), 1.0), ((N, K), K ** -0.5), ((N,), 1.0), ((M, N), 1.0)))
    x = A.double() @ W.double().T + b.double()
    want = {1: 0.5 * x * (1 + torch.erf(x / 2 ** 0.5)), 2: old.double() + x, 3: x}[epi]
    # a sum of K products, each step rounding to 2^-24 of it, a random walk over at most K steps; |gelu'| <= 1.13
    bound = 4 * np.sqrt(K + 16) * 2.0 ** -24 * 1.13 * (A.double().abs() @ W.double().abs().T + b.double().abs() + 1.0)
    Ad, Wd, bd, out = A.cuda(), W.cuda(), b.cuda(), old.cuda()
    B.check(B.lib().zgr_debug_gemm(0, Ad.data_ptr(), Wd.data_ptr(), bd.data_ptr(), out.data_ptr(), epi, M, N, K, torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    assert B.lib().zgr_debug_gemm_form(M, N, K) == (1 if (M, N, K) in PRIVATE else 0)
    off = out.double().cpu() - want
    assert torch.all(off.abs() <= bound)
    if epi == 3:                                                    # the bound above is far from what a random walk leaves: see below
        assert off.norm() <= 2.0 ** -24 * np.sqrt(K / 8) * want.norm()


@pytest.mark.parametrize("M,N,K", [(1024, 1024, 192), (777, 770, 768), (2048, 4096, 32), (2048, 2048, 256), (2048, 2048, 2048), (4096, 1024, 8192)])
@pytest.mark.parametrize("factors", ["gauss", "positive"])
def test_projection_is_as_close_as_fp32_and_unbiased(M, N, K, factors):
    """In the norm, where entry-wise bounds are far above what the planes lose.  Factors of one sign show what they leave out or let fall below the sum's last
    place: nothing averages out.  A sum rounds 6 K / 16 times by at most 2^-24 of its final size (gauss: of its norm over the factors, which the sum's own is)."""
    import torch
    from paper_2601_12917_amd import binding as B
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    draw = torch.randn if factors == "gauss" else lambda *s, **kw: torch.rand(*s, **kw) + 1
    A, W = draw(M, K, generator=gen, device="cuda"), draw(N, K, generator=gen, device="cuda")
    out = torch.empty(M, N, device="cuda")
    B.check(B.lib().zgr_debug_gemm(0, A.data_ptr(), W.data_ptr(), None, out.data_ptr(), 3, M, N, K, torch.cuda.current_stream().cuda_stream))
    want = A.double() @ W.double().T
    off = out.double() - want
    assert off.norm() <= 2.0 ** -24 * np.sqrt(K / 8) * want.norm()              # uniform roundings: 1 / sqrt(3) of their largest
    if K <= 768:                                                                # what is left out averages 2^-38 of a product
        assert abs((off * want.sign()).sum()) <= 0.2 * 2.0 ** -24 * want.abs().sum()


def _wild(x, gen):
    """Entries that are infinite, NaN or close to the largest number, a few in a row of their own each."""
    import torch
    n = x.shape[0]
    for i, v in enumerate((float("inf"), float("-inf"), float("nan"), 3.4e38, -3.3e38, 1e-40)):
        x[(7 * i + 3) % n, int(torch.randint(x.shape[1], (1,), generator=gen))] = v
    x[(7 * 6 + 3) % n, 0], x[(7 * 6 + 3) % n, 1] = float("inf"), float("-inf")
    return x


def _same(got, want):
    """Finite where fp32 is, and the same kind of infinity or NaN where it is not."""
    import torch
    assert torch.equal(torch.isnan(got), torch.isnan(want))
    big = want.abs() > 3.4e38                                       # past the largest fp32 number: sums may or may not reach it on the way
    inf = torch.isinf(want)
    assert torch.equal(got[inf].double(), want[inf])
    ok = ~(torch.isnan(want) | big)
    assert torch.all((got[ok].double() - want[ok]).abs() <= 1e-5 * (1.0 + want[ok].abs()))


@pytest.mark.parametrize("M,N,K,form", [(1024, 1024, 192, 1), (777, 770, 768, 1), (577, 513, 640, 1), (2048, 2048, 256, 0), (577, 513, 256, 4)],
                         ids=["private", "private ragged", "private few", "shared", "product"])
def test_projection_of_wild_operands(M, N, K, form):
    import torch
    from paper_2601_12917_amd import binding as B
    assert B.lib().zgr_debug_gemm_form(M, N, K) == form
    gen = torch.Generator().manual_seed(K)
    A, W = _wild(torch.randn(M, K, generator=gen), gen), torch.randn(N, K, generator=gen).clamp(-3, 3) * 0.01
    want = A.double() @ W.double().T
    Ad, Wd, out = A.cuda(), W.cuda(), torch.zeros(M, N, device="cuda")
    B.check(B.lib().zgr_debug_gemm(0, Ad.data_ptr(), Wd.data_ptr(), None, out.data_ptr(), 3, M, N, K, torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    _same(out.cpu(), want)


@pytest.mark.parametrize("a_k", [1, 0])
@pytest.mark.parametrize("M,N,K", [(231, 1024, 2047), (1024, 1024, 8190), (2048, 4096, 8191)])
@pytest.mark.parametrize("factors", ["gauss", "positive"])
def test_product_with_a_bf16_factor_is_as_close_as_fp32(M, N, K, a_k, factors):
    """Nothing is left out; a sum rounds three times per 32 terms, by at most 2^-24 of its final size, here counted twice.  With factors of one sign the smallest
    planes must not have one."""
    import torch
    from paper_2601_12917_amd import binding as B
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    draw = torch.randn if factors == "gauss" else lambda *s, **kw: torch.rand(*s, **kw) + 1
    A, Bm = draw(M, K, generator=gen, device="cuda"), draw(K, N, generator=gen, device="cuda").bfloat16()
    Ad, out = A if a_k else A.T.contiguous(), torch.empty(M, N, device="cuda")
    B.check(B.lib().zgr_debug_product(Ad.data_ptr(), 0, a_k, Ad.shape[1], 0, Bm.data_ptr(), 1, 0, N, 0, out.data_ptr(), N, 0, M, N, K, 1.0, 1,
                                      None, 0, None, None, 0, torch.cuda.current_stream().cuda_stream))
    want = A.double() @ Bm.double()
    assert (out.double() - want).norm() <= 2.0 ** -24 * np.sqrt(K / 16) * want.norm()


@pytest.mark.parametrize("a_k", [1, 0])
@pytest.mark.parametrize("K", [77, 256])
def test_product_of_wild_operands_with_bf16(a_k, K):
    import torch
    from paper_2601_12917_amd import binding as B
    gen = torch.Generator().manual_seed(K + a_k)
    M, N = 130, 200
    A, Bm = _wild(torch.randn(M, K, generator=gen), gen), (torch.randn(K, N, generator=gen).clamp(-3, 3) * 0.01).bfloat16()
    want = A.double() @ Bm.double()
    Ad, Bd, out = (A if a_k else A.T.contiguous()).cuda(), Bm.cuda(), torch.zeros(M, N, device="cuda")
    sums = None if a_k else torch.zeros(M, device="cuda")
    B.check(B.lib().zgr_debug_product(Ad.data_ptr(), 0, a_k, Ad.shape[1], 0, Bd.data_ptr(), 1, 0, N, 0, out.data_ptr(), N, 0, M, N, K, 1.0, 1,
                                      sums.data_ptr() if sums is not None else None, 0, None, None, 0, torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    _same(out.cpu(), want)
    if sums is not None:
        s = A.double().sum(1)
        assert torch.equal(torch.isnan(sums.cpu()), torch.isnan(s))


def _weight_gradient(dy, u, relu, x, parts):
    """dW, db and dy act'(u) (in place of dy) of zgr_debug_weight_gradient, which has to write every entry."""
    import ctypes as C
    import torch
    from paper_2601_12917_amd import binding as B
    (M, N), K, Mp = dy.shape, x.shape[1], -(-dy.shape[0] // 64) * 64
    dW = [torch.full((N // parts, K), float("nan"), device="cuda") for _ in range(parts)]
    db = [torch.full((N // parts,), float("nan"), device="cuda") for _ in range(parts)]
    scratch = torch.full((6 * N * Mp + 2 * K * Mp + 4 * (N * Mp // 64 + 512),), 0xFF, dtype=torch.uint8, device="cuda")      # NaN, if any of it is read first
    ptrs = lambda t: (C.c_void_p * parts)(*[v.data_ptr() for v in t])
    B.check(B.lib().zgr_debug_weight_gradient(dy.data_ptr(), u.data_ptr() if u is not None else None, relu, x.data_ptr(), M, N, K, parts, ptrs(dW), ptrs(db),
                                              scratch.data_ptr(), scratch.numel(), torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    return torch.cat(dW), torch.cat(db)


@pytest.mark.parametrize("M,N,K,parts", [(1, 64, 64, 1), (63, 192, 64, 3), (65, 1536, 1600, 1), (77, 2112, 2048, 3), (231, 3072, 2048, 3), (130, 5696, 6016, 1), (8191, 128, 192, 2)],
                         ids=lambda v: str(v))
def test_weight_gradient_is_as_close_as_fp32(M, N, K, parts):
    """Each tile size that takes planes (64 x 64, 128 x 128 with one and two blocks a CU), ragged tiles, tokens on either side of a multiple of 64.  Nothing is left
    out; a sum rounds once per 16 terms of a plane, by at most 2^-24 of its size, here counted twice.  GELU's slope in fp32 is within 6 2^-24."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    for draw in (torch.randn, lambda *s, **kw: torch.rand(*s, **kw) + 1):
        dy, x = draw(M, N, generator=gen, device="cuda"), draw(M, K, generator=gen, device="cuda").bfloat16()
        u = torch.randn(M, N, generator=gen, device="cuda") if N % 128 else None
        exact = dy.double()
        if u is not None:
            v = u.double()
            exact = exact * (0.5 * (1 + torch.erf(v / 2 ** 0.5)) + v * torch.exp(-0.5 * v * v) / (2 * np.pi) ** 0.5)
        dW, db = _weight_gradient(dy, u, 0, x, parts)
        if u is not None:
            assert (dy.double() - exact).norm() <= 6 * 2.0 ** -24 * exact.norm()
        want, wb = dy.double().T @ x.double(), dy.double().sum(0)
        assert (dW.double() - want).norm() <= 2.0 ** -24 * np.sqrt(max(M, 16) / 8) * want.norm()
        assert torch.all((db.double() - wb).abs() <= 2.0 ** -24 * 4 * np.sqrt(M + 64) * dy.double().abs().sum(0))


@pytest.mark.parametrize("M", [33, 200])
def test_weight_gradient_of_wild_operands(M):
    import torch
    gen = torch.Generator().manual_seed(M)
    dy, x = _wild(torch.randn(M, 192, generator=gen), gen), (torch.randn(M, 320, generator=gen).clamp(-3, 3) * 0.01).bfloat16()
    want, wb = dy.double().T @ x.double(), dy.double().sum(0)
    dW, db = _weight_gradient(dy.cuda(), None, 0, x.cuda(), 1)
    _same(dW.cpu(), want)
    assert torch.equal(torch.isnan(db.cpu()), torch.isnan(wb))


@pytest.mark.parametrize("M,N,K", [(33, 192, 320), (200, 1600, 1536), (77, 2112, 2048)])
def test_weight_gradient_with_infinite_activations(M, N, K):
    """An infinite entry of x meets the zeros in dy's second and third plane: what fp32 products leave infinite stays infinite, at each tile size that takes planes."""
    import torch
    gen = torch.Generator().manual_seed(M)
    dy, x = torch.randn(M, N, generator=gen).bfloat16().float(), torch.randn(M, K, generator=gen).bfloat16()
    dy[:, ::2] += 2.0 ** -12                                       # every other column with entries in its second plane
    dy[5, 11] = 0.0
    for i, v in ((0, float("inf")), (5, float("-inf")), (9, 3e38), (M - 1, float("nan"))):
        x[i, (37 * i) % K] = v
    want = dy.double().T @ x.double()
    dW, db = _weight_gradient(dy.cuda(), None, 0, x.cuda(), 1)
    _same(dW.cpu(), want)
    assert torch.isinf(dW).sum() > N and torch.all(torch.isfinite(db))
