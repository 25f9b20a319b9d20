"""The fp32 products of the cloud's backward pass (zgr_debug_product) against fp64 on the same values: every layout and storage
type the pass uses, sizes at the edges of the 64 x 64 pieces and the 16-term steps, sums shared by one, four and eight waves and split
over blocks, and the element-by-element form (fewer than four columns, odd bf16 row strides).

A result is a sum of K products rounded to fp32 as it grows: |error| <= (K + parts) 2^-24 sum_k |a||b|, and in practice a
random walk, so the bound asked for is 4 sqrt(K + 16) 2^-24 of that sum of magnitudes."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# (a dtype, a along k, b dtype, b along k)
FORMS = [("f32", 1, "f32", 0), ("f32", 1, "bf16", 0), ("f32", 0, "f32", 0), ("f32", 0, "bf16", 0), ("f32", 1, "f32", 1), ("f32", 1, "bf16", 1), ("bf16", 1, "bf16", 1)]
#        M     N    K  batches pad
SIZES = [(1, 1, 1, 1, 0), (3, 2, 5, 3, 0), (4, 4, 16, 2, 4), (63, 65, 17, 1, 1), (64, 64, 64, 5, 0), (65, 130, 15, 2, 2), (130, 66, 1040, 1, 0), (77, 100, 4100, 1, 4), (5, 36, 35001, 1, 3), (2100, 2050, 40, 1, 6)]


@pytest.mark.parametrize("form", FORMS, ids=lambda f: f"{f[0]}{'k' if f[1] else 'i'}-{f[2]}{'k' if f[3] else 'j'}")
@pytest.mark.parametrize("M,N,K,batches,pad", SIZES)
def test_product_matches_fp64(form, M, N, K, batches, pad):
    import torch
    from paper_2601_12917_amd import binding as B
    a_t, a_k, b_t, b_k = form
    dev = "cuda:0"
    gen = torch.Generator().manual_seed(M * 131 + N * 17 + K + 7 * a_k + b_k)

    def operand(rows, cols, t):                            # [batches, rows, cols + pad], the padding set to what must not be used
        x = torch.randn(batches, rows, cols + pad, generator=gen).to(torch.bfloat16 if t == "bf16" else torch.float32)
        x[:, :, cols:] = float("nan")
        return x.to(dev)
    A = operand(*((M, K) if a_k else (K, M)), a_t)
    Bm = operand(*((N, K) if b_k else (K, N)), b_t)
    ldc = N + pad
    scratch = torch.full((1 << 20,), float("nan"), device=dev)
    ad = A[:, :, :K if a_k else M].double()
    bd = Bm[:, :, :K if b_k else N].double()
    ad, bd = (ad if a_k else ad.transpose(1, 2)).cpu(), (bd.transpose(1, 2) if b_k else bd).cpu()
    want, mag = -0.5 * torch.stack([x @ y for x, y in zip(ad, bd)]), 0.5 * torch.stack([x.abs() @ y.abs() for x, y in zip(ad, bd)])
    for use_scratch in (True, False):
        out = torch.full((batches, M, ldc), 7.0, device=dev)
        out[:, :, :N] = float("nan")                       # every entry has to be written, each time
        sums = torch.full((M,), float("nan"), device=dev) if not a_k and batches == 1 else None
        B.check(B.lib().zgr_debug_product(A.data_ptr(), int(a_t == "bf16"), a_k, A.shape[2], A[0].numel(), Bm.data_ptr(), int(b_t == "bf16"), b_k, Bm.shape[2], Bm[0].numel(),
                                          out.data_ptr(), ldc, M * ldc, M, N, K, -0.5, batches, sums.data_ptr() if sums is not None else None, 0, None,
                                          scratch.data_ptr() if use_scratch else None, scratch.numel() if use_scratch else 0, torch.cuda.current_stream().cuda_stream))
        torch.cuda.synchronize()
        got = out.double().cpu()
        assert torch.all(got[:, :, N:] == 7.0)             # nothing written past a row
        bound = 4 * np.sqrt(K + 16) * 2.0 ** -24
        assert torch.all((got[:, :, :N] - want).abs() <= bound * mag), float(((got[:, :, :N] - want).abs() / mag).max() / bound)
        if sums is not None:
            assert torch.all((sums.double().cpu() - ad[0].sum(1)).abs() <= bound * ad[0].abs().sum(1))


@pytest.mark.parametrize("epilogue", [0, 1, 2, 5], ids=["store", "gelu", "add", "relu"])
@pytest.mark.parametrize("M,N,K", [(5, 7, 12), (33, 95, 200), (70, 190, 1030), (130, 100, 4096), (300, 1100, 260), (2049, 4130, 36)])
def test_product_epilogues(M, N, K, epilogue):
    """The projections of fp32 models: out = act(A W^T + b) or out += A W^T + b, whole and split sums, both piece sizes.  |act'| <= 1.13."""
    import torch
    from paper_2601_12917_amd import binding as B
    dev = "cuda:0"
    gen = torch.Generator().manual_seed(M + N + K)
    A, W, b, old = (torch.randn(*s, generator=gen) * f for s, f in (((M, K), 1.0), ((N, K), K ** -0.5), ((N,), 1.0), ((M, N), 1.0)))
    x = A.double() @ W.double().T + b.double()
    want = {0: x, 1: 0.5 * x * (1 + torch.erf(x / 2 ** 0.5)), 2: old.double() + x, 5: x.clamp(min=0)}[epilogue]
    bound = 4 * np.sqrt(K + 16) * 2.0 ** -24 * 1.13 * (A.double().abs() @ W.double().abs().T + b.double().abs() + 1.0)
    Ad, Wd, bd = A.to(dev), W.to(dev), b.to(dev)
    scratch = torch.full((1 << 21,), float("nan"), device=dev)
    for n in (scratch.numel(), 0):
        out = old.to(dev).clone()
        B.check(B.lib().zgr_debug_product(Ad.data_ptr(), 0, 1, K, 0, Wd.data_ptr(), 0, 1, K, 0, out.data_ptr(), N, 0, M, N, K, 1.0, 1, None, epilogue, bd.data_ptr(),
                                          scratch.data_ptr() if n else None, n, torch.cuda.current_stream().cuda_stream))
        torch.cuda.synchronize()
        assert torch.all((out.double().cpu() - want).abs() <= bound)
