"""The general dense update where its split changes: 4 or 16 waves on one row tile, one wave per tile, groups of 64 columns; sizes
around the tiles.  Compared with fp64 torch, relative to the sum of the absolute terms; 1e-5, the bar of fp32 sums."""
import pytest
import torch

from paper_2412_12218_amd import binding as B

pytestmark = pytest.mark.gpu
F32, F16, BF16 = torch.float32, torch.float16, torch.bfloat16


@pytest.mark.parametrize("dtype", [F32, F16, BF16])
@pytest.mark.parametrize("n,d_in,d_out", [(1, 513, 7), (17, 512, 16), (8192, 1025, 33), (8193, 1025, 33), (100, 511, 64), (33, 2049, 64),
                                          (16384, 37, 65), (16385, 37, 65), (16400, 300, 130), (16391, 70, 128)])
def test_update_gemm_at_the_lines_of_its_split(dtype, n, d_in, d_out):
    gen = torch.Generator(device="cuda").manual_seed(n + d_in)
    X = torch.randn((n, d_in + 1), generator=gen, device="cuda").to(dtype)[:, 1:]  # rows at the alignment of an element
    W = torch.randn((d_in, d_out), generator=gen, device="cuda").to(dtype)
    scale = torch.rand(n, generator=gen, device="cuda") + 0.5
    ref, terms = X.double() @ W.double(), X.double().abs() @ W.double().abs()
    out = torch.full((n, d_out + 3), 7.0, device="cuda")
    Z = B.ftc_update_gemm(X, W, out=out[:, :d_out], relu=True, row_scale=scale)
    s = scale.double()[:, None]
    assert float(((Z.double() - (ref * s).clamp(min=0)).abs() / (terms * s)).max()) <= 1e-5
    assert torch.all(out[:, d_out:] == 7.0)


@pytest.mark.parametrize("n", [380_000, 401_003])
@pytest.mark.parametrize("d_out", [65, 128, 130, 200])
def test_update_gemm_of_rows_read_more_than_once(n, d_out):
    """fp32, 130 columns: groups of 64 output columns below 300 MB, above it of 128 where these need no padding."""
    test_update_gemm_at_the_lines_of_its_split(F32, n, 130, d_out)
