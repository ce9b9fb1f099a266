"""Dense products of few rows, the contraction split over the waves of a workgroup: edges of its tiles and steps, the lines of its
dispatch, numbers that can't be taken in bf16 pieces.  Compared with fp64 torch, relative to the sum of the absolute terms.  A wave
rounds once per 32 terms, the waves' sums are added up (16 / 4 + 2 roundings), the terms are exact or, in pieces, short of 2^-24 of
themselves: (d_in / 16 + 8) 2^-24 is twice that."""
import pytest
import torch

from paper_2412_12218_amd import binding as B

pytestmark = pytest.mark.gpu
F32, F16, BF16 = torch.float32, torch.float16, torch.bfloat16


def check(X, W, relu=False, scale=None):
    n, d_in, d_out = X.shape[0], X.shape[1], W.shape[1]
    out = torch.full((n, d_out + 2), 7.0, device="cuda")
    Z = B.ftc_update_gemm(X, W, out=out[:, 1:d_out + 1], relu=relu, row_scale=scale)
    ref, terms = X.double() @ W.double(), X.double().abs() @ W.double().abs()
    if scale is not None:
        ref, terms = ref * scale.double()[:, None], terms * scale.double()[:, None]
    if relu:
        ref = ref.clamp(min=0)
    assert float(((Z.double() - ref).abs() / terms.clamp(min=1e-300)).max()) <= (d_in / 16 + 8) * 2.0 ** -24
    assert torch.all(out[:, 0] == 7.0) and torch.all(out[:, d_out + 1] == 7.0)


@pytest.mark.parametrize("dtype", [F32, F16, BF16])
@pytest.mark.parametrize("n,d_in,d_out", [
    (1, 1, 1), (16, 32, 16), (17, 31, 17), (15, 33, 33), (100, 127, 15), (1000, 129, 22), (2708, 511, 47), (2708, 512, 32), (2708, 513, 64),
    (1024, 1433, 16), (4096, 1433, 7), (4097, 640, 33), (300, 2047, 65), (300, 2081, 130), (6144, 40, 65), (6145, 40, 65), (8192, 31, 40),
    (8193, 31, 40), (12288, 65, 64), (12289, 65, 64), (12289, 33, 66), (16384, 33, 16), (16385, 33, 16)])
def test_rows_at_the_alignment_of_an_element(dtype, n, d_in, d_out):
    gen = torch.Generator(device="cuda").manual_seed(n + d_in + d_out)
    buf = torch.full((n, d_in + 3), float("nan"), device="cuda", dtype=dtype)  # nothing beside the rows is used
    buf[:, 1:d_in + 1] = torch.randn((n, d_in), generator=gen, device="cuda").to(dtype)
    check(buf[:, 1:d_in + 1], torch.randn((d_in, d_out), generator=gen, device="cuda").to(dtype))


@pytest.mark.parametrize("dtype", [F32, F16, BF16])
@pytest.mark.parametrize("n,d_in,d_out", [(4096, 16, 16), (4097, 16, 16), (8192, 32, 7), (8193, 32, 7), (16384, 64, 64), (16385, 64, 64),
                                          (500, 256, 64), (500, 264, 64), (777, 12, 8), (777, 16, 8), (777, 16, 12), (16385, 32, 8),
                                          (777, 3, 40), (16385, 4, 130), (100_001, 2, 16)])
def test_aligned_rows_with_the_epilogue(dtype, n, d_in, d_out):
    gen = torch.Generator(device="cuda").manual_seed(n + d_in + d_out)
    X = torch.randn((n, d_in), generator=gen, device="cuda").to(dtype)
    check(X, torch.randn((d_in, d_out), generator=gen, device="cuda").to(dtype), relu=True,
          scale=torch.rand(n, generator=gen, device="cuda") + 0.5)


@pytest.mark.parametrize("dtype", [F32, F16])
@pytest.mark.parametrize("d_in", [70, 530])
def test_infinities_and_nan(dtype, d_in):
    """Of X and of W, in whole steps and in the last one: what fp32 arithmetic makes of them."""
    gen = torch.Generator().manual_seed(d_in)
    n, d_out = 300, 20
    X, W = torch.randn((n, d_in), generator=gen).to(dtype), torch.randn((d_in, d_out), generator=gen).to(dtype)
    X[3, 2], X[40, d_in - 1], X[70, 0] = float("inf"), float("-inf"), float("nan")
    W[2, 3], W[d_in - 1, 4] = 0.0, 0.0  # infinity times zero
    for W1 in (W, torch.where((torch.arange(d_out) == 5) & (torch.arange(d_in) == d_in - 1)[:, None], torch.full_like(W, float("inf")), W)):
        ref = X.double() @ W1.double()
        got = B.ftc_update_gemm(X.cuda(), W1.cuda()).cpu()
        assert torch.equal(torch.isnan(got), torch.isnan(ref)) and torch.equal(torch.isposinf(got), torch.isposinf(ref))
        assert torch.equal(torch.isneginf(got), torch.isneginf(ref))
        ok = torch.isfinite(ref)
        terms = (X.double().abs() @ W1.double().abs())[ok]
        assert float(((got.double()[ok] - ref[ok]).abs() / terms).max()) <= 1e-5  # (fp32: a sum of d_in terms, one after the other)


@pytest.mark.parametrize("dtype", [F32, F16, BF16])
@pytest.mark.parametrize("n,d_in,d_out", [(1, 1, 65), (17, 33, 65), (500, 300, 300), (2731, 96, 96), (4096, 64, 66), (4097, 64, 66), (2708, 7, 504), (13_107, 20, 129)])
def test_input_gradient_of_few_results(dtype, n, d_in, d_out):
    """dX = G W^T of a contraction of more than 64 columns: the rows of W are read eight elements at a time, or one by one in the last step."""
    gen = torch.Generator(device="cuda").manual_seed(n + d_in)
    X = torch.randn((n, d_in), generator=gen, device="cuda").to(dtype)
    W = torch.randn((d_in, d_out), generator=gen, device="cuda").to(dtype)
    G = torch.randn((n, d_out + 1), generator=gen, device="cuda")[:, 1:]
    dX = torch.full((n, d_in + 2), 7.0, device="cuda")
    B.ftc_update_gemm_backward(X, W, G, dX=dX[:, 1:d_in + 1])
    ref, terms = G.double() @ W.double().T.contiguous(), G.double().abs() @ W.double().abs().T.contiguous()
    assert float(((dX[:, 1:d_in + 1].double() - ref).abs() / terms.clamp(min=1e-300)).max()) <= (d_out / 16 + 8) * 2.0 ** -24
    assert torch.all(dX[:, 0] == 7.0) and torch.all(dX[:, d_in + 1] == 7.0)
