"""Dense products of any width and alignment on the 16-bit matrix cores: edges of the tiles and chunks, the lines of their
dispatch, numbers that can't be taken in bf16 pieces, and dX = G W^T.  Compared with fp64 torch, relative to the sum of the
absolute terms.  A sum is rounded once per 32 terms (16 bits: a quarter of that and once per 128), the terms are exact or, in
pieces, short of 2^-24 of themselves: (d_in / 16 + 8) 2^-24 is twice that."""
import pytest
import torch

from paper_2412_12218_amd import binding as B

pytestmark = pytest.mark.gpu
F32, F16, BF16 = torch.float32, torch.float16, torch.bfloat16


def bound(d_in):
    return (d_in / 16 + 8) * 2.0 ** -24


def rel(Z, X, W):
    ref, terms = X.double() @ W.double(), X.double().abs() @ W.double().abs()
    return float(((Z.double() - ref).abs() / terms.clamp(min=1e-300)).max())


@pytest.mark.parametrize("dtype", [F32, F16, BF16])
@pytest.mark.parametrize("n,d_in,d_out", [
    (1, 1, 65), (15, 31, 66), (65, 32, 80), (64, 33, 128), (1000, 63, 129), (4096, 127, 64), (4097, 127, 7), (4097, 64, 33),
    (8193, 128, 33), (12288, 65, 17), (12289, 65, 17), (16385, 129, 16), (98303, 17, 16), (98304, 17, 16), (98305, 70, 3), (65535, 70, 9), (65536, 70, 9), (65537, 200, 16), (98304, 70, 16), (98305, 200, 7), (114688, 65, 16), (114689, 70, 10),
    (65535, 40, 100), (65536, 40, 200), (131073, 20, 40), (5000, 641, 65), (20001, 257, 48)])
def test_update_gemm_at_edges_of_tiles_and_chunks(dtype, n, d_in, d_out):
    gen = torch.Generator(device="cuda").manual_seed(n + d_in + d_out)
    buf = torch.full((n, d_in + 3), float("nan"), device="cuda", dtype=dtype)  # rows at the alignment of an element, nothing beside them is used
    buf[:, 1:d_in + 1] = torch.randn((n, d_in), generator=gen, device="cuda").to(dtype)
    X = buf[:, 1:d_in + 1]
    W = torch.randn((d_in, d_out), generator=gen, device="cuda").to(dtype)
    out = torch.full((n, d_out + 2), 7.0, device="cuda")
    Z = B.ftc_update_gemm(X, W, out=out[:, 1:d_out + 1])
    assert rel(Z, X, W) <= bound(d_in)
    assert torch.all(out[:, 0] == 7.0) and torch.all(out[:, d_out + 1] == 7.0)


@pytest.mark.parametrize("dtype", [F16, BF16])
@pytest.mark.parametrize("n,d_in,d_out", [(65_535, 256, 65), (65_536, 255, 65), (65_536, 256, 65), (65_537, 257, 128), (65_600, 384, 129), (70_001, 513, 200), (98_303, 300, 33),
                                          (98_304, 256, 33), (98_305, 385, 64), (100_001, 1433, 40), (300_001, 256, 48), (300_001, 256, 500), (65_791, 700, 64 * 33)])
def test_long_16_bit_rows_in_tiles_of_four_and_two_a_wave(dtype, n, d_in, d_out):
    """Rows, columns and chunks that end inside a tile, a step and a half chunk; W staged once and per chunk."""
    test_update_gemm_at_edges_of_tiles_and_chunks(dtype, n, d_in, d_out)


@pytest.mark.parametrize("dtype", [F16, BF16])
@pytest.mark.parametrize("n,d_in,d_out", [(65_537, 264, 130), (98_311, 520, 40), (65_536, 192, 65), (70_001, 184, 65), (70_001, 248, 129)])
def test_long_16_bit_rows_scaled_and_clipped_in_aligned_rows(dtype, n, d_in, d_out):
    gen = torch.Generator(device="cuda").manual_seed(n)
    X, W = torch.randn((n, d_in), generator=gen, device="cuda").to(dtype), torch.randn((d_in, d_out), generator=gen, device="cuda").to(dtype)
    scale = torch.rand((n,), generator=gen, device="cuda") + 0.5
    X[5, 7], X[n - 1, d_in - 1] = float("inf"), float("nan")
    Z = B.ftc_update_gemm(X, W, row_scale=scale, relu=True, out=torch.empty((n, d_out), device="cuda"))
    ref, terms = X.double() @ W.double() * scale.double()[:, None], X.double().abs() @ W.double().abs() * scale.double()[:, None]
    ok = torch.ones(n, dtype=torch.bool, device="cuda")
    ok[5] = ok[n - 1] = False
    assert float(((Z.double() - ref.clamp(min=0))[ok].abs() / terms[ok]).max()) <= bound(d_in) + 2.0 ** -23
    assert torch.equal(torch.isposinf(Z[5]), torch.isposinf(ref[5]))


@pytest.mark.parametrize("n,d_in,d_out", [(6144, 8, 85), (6144, 8, 86), (1048, 32, 500), (1049, 32, 500), (1049, 48, 500), (1049, 49, 500), (6144, 5, 500), (6143, 33, 131)])
def test_one_and_two_steps_of_the_contraction_on_both_sides_of_their_line(n, d_in, d_out):
    test_update_gemm_at_edges_of_tiles_and_chunks(F32, n, d_in, d_out)


@pytest.mark.parametrize("d_in", [8, 48])
def test_products_of_one_and_two_steps_take_the_same_time_on_both_sides_of_the_line_of_few_rows(d_in):
    """6144 and 6145 rows of 8 and 48 fp32 elements into 500 columns: twice the time where one or two waves of four had work."""
    times = []
    for n in (6144, 6145):
        X, W, out = torch.randn((n, d_in), device="cuda"), torch.randn((d_in, 500), device="cuda"), torch.empty((n, 500), device="cuda")
        times.append(us(lambda: B.ftc_update_gemm(X, W, out=out)))
    print("us", times)
    assert times[0] <= 1.6 * times[1]


def test_a_few_columns_beyond_a_group_do_not_cost_a_group():
    """16-bit rows of 512 elements into 129 columns next to 128: twice as long when the second group took all 128 columns' time."""
    X = torch.randn((400_000, 512), device="cuda").to(F16)
    times = []
    for d in (128, 129):
        W, out = torch.randn((512, d), device="cuda").to(F16), torch.empty((400_000, d), device="cuda", dtype=F16)
        times.append(us(lambda: B.ftc_update_gemm(X, W, out=out)))
    print("us", times)
    assert times[1] <= 1.6 * times[0]


@pytest.mark.parametrize("n,d_in,d_out", [(300, 70, 70), (20000, 33, 20)])
def test_numbers_that_bf16_pieces_cannot_hold(n, d_in, d_out):
    """Infinities, NaN, the largest and the smallest numbers: what fp32 arithmetic makes of them."""
    gen = torch.Generator().manual_seed(1)
    X, W = torch.randn((n, d_in), generator=gen), torch.randn((d_in, d_out), generator=gen)
    X[3, 2], X[5, d_in - 1], X[70, 0], X[71, 1], X[200, 7] = float("inf"), float("-inf"), float("nan"), 3.4e38, 3.3961775e38
    X[90:110] *= 1e-38  # subnormal, or pieces of them are
    W[2, 3] = 0.0       # infinity times zero
    for W1 in (W, torch.where(torch.arange(d_out) == 4, W * float("inf"), W), torch.where(torch.arange(d_out) == 5, W * 1e-39, W)):
        ref = X @ W1
        got = B.ftc_update_gemm(X.cuda(), W1.cuda()).cpu()
        assert torch.equal(torch.isnan(got), torch.isnan(ref)) and torch.equal(torch.isposinf(got), torch.isposinf(ref))
        assert torch.equal(torch.isneginf(got), torch.isneginf(ref))
        ok = torch.isfinite(ref) & (ref.abs() > 1e-30)
        terms = X.double().abs() @ W1.double().abs()
        err = ((got.double() - X.double() @ W1.double()).abs() / terms)[ok & torch.isfinite(terms)]
        assert float(err.max()) <= 1e-5  # a sum of d_in terms in fp32, one after the other
        small = ref[90:110].double().abs()
        live = (small > 1e-37) & torch.isfinite(terms[90:110])
        assert float(((got[90:110].double() - X[90:110].double() @ W1.double()).abs() / terms[90:110])[live].max()) <= 1e-5


@pytest.mark.parametrize("dtype", [F32, F16, BF16])
@pytest.mark.parametrize("n,d_in,d_out", [(1, 1, 1), (63, 17, 5), (1000, 16, 22), (4000, 33, 64), (777, 128, 65), (300, 130, 130), (70_001, 65, 8)])
def test_input_gradient_at_edges_of_tiles_and_chunks(dtype, n, d_in, d_out):
    gen = torch.Generator(device="cuda").manual_seed(n + d_in)
    X = torch.randn((n, d_in), generator=gen, device="cuda").to(dtype)
    W = torch.randn((d_in, d_out), generator=gen, device="cuda").to(dtype)
    G = torch.randn((n, d_out + 1), generator=gen, device="cuda")[:, 1:]
    dX = torch.full((n, d_in + 1), 7.0, device="cuda")
    B.ftc_update_gemm_backward(X, W, G, dX=dX[:, :d_in])
    assert rel(dX[:, :d_in], G, W.T) <= bound(d_out)
    assert torch.all(dX[:, d_in] == 7.0)


@pytest.mark.parametrize("dtype", [F32, F16, BF16])
@pytest.mark.parametrize("n,d_in,d_out", [(4097, 65, 32), (9000, 66, 64), (4100, 64, 96), (10_001, 40, 131), (20_000, 130, 300), (70_001, 129, 1), (65, 1433, 40),
                                          (3000, 1700, 7), (327_679, 65, 3), (327_680, 65, 3), (327_680, 65, 9), (70_001, 130, 5), (4097, 17, 8), (1000, 65, 9),
                                          (700_001, 91, 8), (700_001, 91, 13), (700_001, 91, 17), (1_200_001, 91, 16), (1_200_001, 91, 17), (400_001, 330, 9), (500_009, 128, 3)])
def test_input_gradient_of_whole_and_cut_chunks_of_w(dtype, n, d_in, d_out):
    """Rows of W are read eight elements at a time where the chunk is whole, else one by one; X and W of each type.  Several groups of
    64 columns of dX: a workgroup each on neighbouring places up to 327 679 rows, in walks of 1024 / groups or 40 workgroups a group.  Above 250 MB
    from up to 8 columns, 350 MB from up to 16: whole rows."""
    test_input_gradient_at_edges_of_tiles_and_chunks(dtype, n, d_in, d_out)


@pytest.mark.parametrize("dtype", [F32, F16, BF16])
@pytest.mark.parametrize("n,d_in,d_out", [(32768, 33, 33), (32769, 64, 64), (32800, 65, 129), (65536, 128, 128), (65537, 129, 200), (70_003, 300, 65),
                                          (33_000, 130, 47), (40_000, 1030, 65)])
def test_weight_gradient_at_edges_of_tiles_and_steps(dtype, n, d_in, d_out):
    """Rows in steps of 32, a sum of shares: 2 n / 32 / shares + shares / 4 + 8 roundings (at least 64 shares here), the terms are exact."""
    gen = torch.Generator(device="cuda").manual_seed(n + d_in)
    buf = torch.full((n, d_in + 2), float("nan"), device="cuda", dtype=dtype)
    buf[:, 1:d_in + 1] = torch.randn((n, d_in), generator=gen, device="cuda").to(dtype)
    X, G = buf[:, 1:d_in + 1], torch.randn((n, d_out + 1), generator=gen, device="cuda")[:, 1:]
    W = torch.zeros((d_in, d_out), device="cuda", dtype=dtype)
    for Z in (None, torch.randn((n, d_out), generator=gen, device="cuda"), torch.randn((n, d_out), generator=gen, device="cuda").to(F16)):
        masked = G if Z is None else torch.where(Z > 0, G, torch.zeros_like(G))
        dW = B.ftc_update_gemm_backward(X, W, G, Z=Z, want_dX=False)[1]
        ref, terms = X.double().T @ masked.double(), X.double().abs().T @ masked.double().abs()
        assert float(((dW.double() - ref).abs() / terms).max()) <= (2 * n / 32 / 64 + 64) * 2.0 ** -24


@pytest.mark.parametrize("dtype", [F32, F16, BF16])
@pytest.mark.parametrize("n,d_in,d_out", [(100_001, 64, 64), (200_001, 33, 50), (100_003, 300, 33), (66_000, 128, 60), (100_003, 97, 40), (33_001, 500, 48),
                                          (45_000, 128, 128), (65_600, 65, 65), (33_000, 200, 200), (100_000, 200, 136)])
def test_weight_gradient_by_tiles_of_each_size(dtype, n, d_in, d_out):
    """Three each that go to 4 x 4, 8 x 4 and 8 x 8 tiles of 16 columns; the last, in fp32, to two launches of the other kernel."""
    test_weight_gradient_at_edges_of_tiles_and_steps(dtype, n, d_in, d_out)


@pytest.mark.parametrize("dtype", [F32, F16, BF16])
@pytest.mark.parametrize("n,d_in,d_out", [(32_800, 40, 70), (100_001, 40, 64), (66_000, 128, 60), (45_000, 100, 128)])
def test_weight_gradient_of_numbers_that_bf16_pieces_cannot_hold(dtype, n, d_in, d_out):
    """By the fp32 kernel, and by 4 x 4, 8 x 4 and 8 x 8 tiles."""
    gen = torch.Generator().manual_seed(2)
    X, G = torch.randn((n, d_in), generator=gen).to(dtype), torch.randn((n, d_out), generator=gen)
    X[100, 3], X[5000, 39], G[7, 1], G[n - 1, d_out - 1], G[40, 5] = float("inf"), float("nan"), float("-inf"), float("nan"), 3.4e38
    X[40] = 0.5
    G[300:310] *= 1e-38
    X[7, 2] = 0.0  # infinity times zero
    ref = X.double().T @ G.double()
    dW = B.ftc_update_gemm_backward(X.cuda(), torch.zeros((d_in, d_out), dtype=dtype).cuda(), G.cuda(), want_dX=False)[1].cpu()
    assert torch.equal(torch.isnan(dW), torch.isnan(ref)) and torch.equal(torch.isinf(dW), torch.isinf(ref))
    assert torch.equal(dW > 0, ref.float() > 0)
    terms = X.double().abs().T @ G.double().abs()
    ok = torch.isfinite(terms)
    assert float(((dW.double() - ref).abs() / terms)[ok].max()) <= 1e-5


@pytest.mark.parametrize("dtype", [F32, F16, BF16])
@pytest.mark.parametrize("column", [0, -1])
def test_weight_gradient_of_an_infinity_in_the_first_step_of_every_share(dtype, column):
    """Row 31 of every 32 rows is loaded by the last wave, row 0 by the first: whichever wave finds the infinity, the step is not taken in pieces."""
    gen = torch.Generator().manual_seed(3)
    n, d_in, d_out = 100_000, 48, 64
    X, G = (torch.rand((n, d_in), generator=gen) + 0.5).to(dtype).cuda(), torch.randn((n, d_out), generator=gen).cuda()
    G[31 if column else 0::32, column] = float("inf")
    dW = B.ftc_update_gemm_backward(X, torch.zeros((d_in, d_out), dtype=dtype).cuda(), G, want_dX=False)[1]
    assert torch.isposinf(dW[:, column]).all() and int(torch.isfinite(dW).sum()) == d_in * (d_out - 1)


def us(f):
    """Least time of a call over five batches."""
    for _ in range(3):
        f()
    best = float("inf")
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(10):
            f()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) * 100)
    return best


@pytest.mark.parametrize("kind,n,d_in,d_out", [("update", 100_000, 300, 128), ("update", 100_000, 1433, 16), ("update", 2708, 1433, 64), ("update", 8000, 301, 64),
                                               ("dX", 100_000, 300, 128), ("dX", 2708, 64, 504), ("dW", 100_000, 300, 128), ("dW", 66_000, 128, 60)])
def test_small_numbers_cost_the_fp32_instruction_and_no_more(kind, n, d_in, d_out):
    """A number that bf16 pieces can't hold in one place of W, or in one row of 16 (dW: 32): the tiles (dW: steps) it is in by the fp32
    instruction from memory, about as long as that kernel alone took, and the pieces before.  (One term after the other: 20 to 100 times.)"""
    gen = torch.Generator(device="cuda").manual_seed(n)
    X, G = torch.randn((n, d_in), generator=gen, device="cuda"), torch.randn((n, d_out), generator=gen, device="cuda")
    W = torch.randn((d_in, d_out), generator=gen, device="cuda")
    out, dX = torch.empty((n, d_out), device="cuda"), torch.empty((n, d_in), device="cuda")

    def run():
        if kind == "update":
            B.ftc_update_gemm(X, W, out=out)
        elif kind == "dX":
            B.ftc_update_gemm_backward(X, W, G, dX=dX)
        else:
            B.ftc_update_gemm_backward(X, W, G, want_dX=False)
    plain = us(run)
    A = X if kind == "update" else G
    times = []
    if kind != "dW":
        W[d_in // 2, d_out // 2] = 1.2345679e-36
        times.append(us(run))
        W[d_in // 2, d_out // 2] = 1.0
    A[5::16 if kind != "dW" else 32, 3] = 1.2345679e-36
    times.append(us(run))
    print(kind, n, d_in, d_out, "us", plain, times)
    assert max(times) <= 4 * plain


@pytest.mark.parametrize("n,d_in,d_out", [(20_000, 64, 64), (20_000, 63, 33), (100_000, 200, 16), (20_000, 200, 70), (300, 70, 70), (2708, 504, 33)])
def test_small_numbers_in_any_step(n, d_in, d_out):
    """Columns of W, rows of X and rows of W (in dX: columns) that bf16 pieces can't hold, in each step: rounded no more than once per four terms."""
    gen = torch.Generator(device="cuda").manual_seed(n + d_in)
    for k in range(5, d_in, 32):
        X, W = torch.randn((n, d_in), generator=gen, device="cuda"), torch.randn((d_in, d_out), generator=gen, device="cuda")
        W[:, d_out // 2] *= 1e-33
        W[k, 0] = 1e-34
        X[n // 2 + k % 16] *= 1e-3
        X[3::64, k] = 1e-33
        Z = B.ftc_update_gemm(X, W)
        assert rel(Z, X, W) <= (d_in / 4 + 8) * 2.0 ** -24
        dX = torch.empty((n, d_out), device="cuda")  # X as the gradient of a product with W^T
        B.ftc_update_gemm_backward(torch.empty((n, d_out), device="cuda"), W.T.contiguous(), X, dX=dX)
        assert rel(dX, X, W) <= (d_in / 4 + 8) * 2.0 ** -24


@pytest.mark.parametrize("dtype", [F32, F16])
@pytest.mark.parametrize("n,d_in,d_out", [(20_000, 1, 70), (20_000, 2, 33), (100_001, 1, 3), (100_000, 2, 200), (300, 1, 20), (5000, 2, 64), (33, 2, 7), (6000, 1, 130)])
def test_sums_of_one_and_two_products_are_rounded_once_and_twice(dtype, n, d_in, d_out):
    """Half a unit in the last place of the product, or of one of the products and of the sum: what fused multiply-adds leave."""
    gen = torch.Generator(device="cuda").manual_seed(n + d_in)
    X, W = torch.randn((n, d_in), generator=gen, device="cuda"), torch.randn((d_in, d_out), generator=gen, device="cuda")
    Wt = W.T.to(dtype)  # the gradient's weights may be of another type
    dX = torch.full((n, d_out + 1), 7.0, device="cuda")
    B.ftc_update_gemm_backward(torch.zeros((n, d_out), device="cuda", dtype=dtype), Wt.contiguous(), X, dX=dX[:, :d_out])
    assert torch.all(dX[:, d_out] == 7.0)
    for Z, W1 in ((B.ftc_update_gemm(X, W), W), (dX[:, :d_out], Wt.float().T)):
        terms = X.double()[:, :, None] * W1.double()[None]
        ref = terms.sum(1)
        allowed = ref.abs() + (terms.abs().amax(1) if d_in == 2 else 0.0)
        assert float(((Z.double() - ref).abs() / allowed).max()) <= 2.0 ** -24 * (1 + 2.0 ** -20)


@pytest.mark.parametrize("n,d_in,d_out", [(20_000, 3, 70), (20_000, 4, 16), (300, 3, 20), (5000, 4, 64), (20_000, 5, 16), (300, 5, 20)])
def test_infinities_and_nan_in_sums_of_few_products(n, d_in, d_out):
    gen = torch.Generator().manual_seed(d_in)
    X, W = torch.randn((n, d_in), generator=gen), torch.randn((d_in, d_out), generator=gen)
    X[3, 2], X[40, d_in - 1], X[70, 0], W[d_in - 1, 4], W[2, 5] = float("inf"), float("-inf"), float("nan"), 0.0, float("inf")
    X[90:110] *= 1e-36
    ref = X.double() @ W.double()
    dX = torch.empty((n, d_out), device="cuda")
    B.ftc_update_gemm_backward(torch.zeros((n, d_out), device="cuda"), W.T.contiguous().cuda(), X.cuda(), dX=dX)
    for got in (B.ftc_update_gemm(X.cuda(), W.cuda()).cpu(), dX.cpu()):
        assert torch.equal(torch.isnan(got), torch.isnan(ref)) and torch.equal(torch.isposinf(got), torch.isposinf(ref))
        ok = torch.isfinite(ref)
        terms = (X.double().abs() @ W.double().abs())[ok]
        assert float(((got.double()[ok] - ref[ok]).abs() / terms).max()) <= d_in * 2.0 ** -24 * (1 + 2.0 ** -20)


LARGE = 1.998046875 * 2.0 ** 63  # its first bf16 piece is 2^64


@pytest.mark.parametrize("n,d_in,d_out", [(20_000, 70, 70), (100_000, 33, 9), (100_000, 100, 16), (300, 70, 20), (2708, 504, 64), (20_000, 33, 20)])
def test_products_and_sums_below_the_largest_number_are_finite(n, d_in, d_out):
    """One product, and a sum of two, of 0.999 times the largest number, whose bf16 pieces make infinity."""
    gen = torch.Generator(device="cuda").manual_seed(n)
    X, W = torch.randn((n, d_in), generator=gen, device="cuda"), torch.randn((d_in, d_out), generator=gen, device="cuda")
    W[d_in - 1, 2], W[3, 2], W[9, 2] = 2.0 ** 64, 2.0 ** 63, 2.0 ** 63
    X[5], X[n - 1], X[7] = 0.0, 0.0, 0.0
    X[:, 3], X[:, 9], X[:, d_in - 1] = 0.0, 0.0, 0.0
    X[5, d_in - 1], X[n - 1, 3], X[n - 1, 9], X[7, d_in - 1] = LARGE, LARGE, LARGE, -LARGE
    X[9, 3] = float("inf")
    dX = torch.empty((n, d_out), device="cuda")
    B.ftc_update_gemm_backward(torch.zeros((n, d_out), device="cuda"), W.T.contiguous(), X, dX=dX)
    for Z in (B.ftc_update_gemm(X, W), dX):
        assert Z[5, 2] == LARGE * 2.0 ** 64 and Z[n - 1, 2] == LARGE * 2.0 ** 64 and Z[7, 2] == -LARGE * 2.0 ** 64
        assert torch.isinf(Z[9]).all()
        Z[9] = 0.0
        X1 = X.clone()
        X1[9] = 0.0
        assert rel(Z, X1, W) <= (d_in / 4 + 8) * 2.0 ** -24


@pytest.mark.parametrize("dtype", [F32, F16, BF16])
@pytest.mark.parametrize("n,d_in,d_out", [(32_800, 40, 70), (100_001, 40, 64), (66_000, 128, 60), (45_000, 100, 128)])
def test_weight_gradients_below_the_largest_number_are_finite(dtype, n, d_in, d_out):
    gen = torch.Generator(device="cuda").manual_seed(n)
    X, G = torch.randn((n, d_in), generator=gen, device="cuda").to(dtype), torch.randn((n, d_out), generator=gen, device="cuda")
    rows = [n // 3, n - 1]
    X[rows], G[rows] = 0.0, 0.0
    X[:, 3], G[:, 2], G[:, 4] = 0.0, 0.0, 0.0
    X[rows[0], 3], G[rows[0], 2] = 2.0 ** 14, LARGE * 2.0 ** 50
    X[rows[1], 3], G[rows[1], 4] = 2.0 ** 14, -LARGE * 2.0 ** 50
    for masked in (False, True):
        Z = torch.ones((n, d_out), device="cuda") if masked else None
        dW = B.ftc_update_gemm_backward(X, torch.zeros((d_in, d_out), dtype=dtype, device="cuda"), G, Z=Z, want_dX=False)[1]
        assert dW[3, 2] == LARGE * 2.0 ** 64 and dW[3, 4] == -LARGE * 2.0 ** 64
        ref, terms = X.double().T @ G.double(), X.double().abs().T @ G.double().abs()
        assert float(((dW.double() - ref).abs() / terms.clamp(min=1e-300)).max()) <= 1e-5


@pytest.mark.parametrize("dtype,k", [(F32, 3), (F32, 9), (BF16, 70), (F16, 2)])
def test_more_columns_than_a_launch_takes(dtype, k):
    """65 535 groups of 64 columns and more, forward and in the input gradient."""
    gen = torch.Generator(device="cuda").manual_seed(k)
    n, d = 3, 65_535 * 64 + 1000
    X, W = torch.randn((n, k), generator=gen, device="cuda").to(dtype), torch.randn((k, d), generator=gen, device="cuda").to(dtype)
    assert rel(B.ftc_update_gemm(X, W), X, W) <= bound(k)
    dX = torch.empty((n, d), device="cuda")
    G = X.float()
    B.ftc_update_gemm_backward(torch.zeros((n, d), device="cuda", dtype=dtype), W.T.contiguous(), G, dX=dX)
    assert rel(dX, G, W) <= bound(k)


@pytest.mark.parametrize("dtype", [F16, BF16])
@pytest.mark.parametrize("n,d_in,d_out", [(20_000, 70, 3), (5000, 200, 8), (700_001, 200, 7), (700_001, 201, 12), (20_000, 70, 40)])
def test_input_gradient_in_16_bits(dtype, n, d_in, d_out):
    """The same as in 32 bits, rounded once; a contraction of few indices, whole rows above 250 MB, tiles."""
    gen = torch.Generator(device="cuda").manual_seed(n + d_in)
    X, W = torch.zeros((n, d_in), device="cuda", dtype=dtype), torch.randn((d_in, d_out), generator=gen, device="cuda").to(dtype)
    G = torch.randn((n, d_out), generator=gen, device="cuda")
    dX = torch.full((n, d_in + 3), 7.0, device="cuda", dtype=dtype)
    B.ftc_update_gemm_backward(X, W, G, dX=dX[:, :d_in])
    ref = G.double() @ W.double().T.contiguous()
    eps = 2.0 ** (-11 if dtype == F16 else -8)
    terms = G.double().abs() @ W.double().abs().T.contiguous()
    assert bool(((dX[:, :d_in].double() - ref).abs() <= eps * ref.abs() + bound(d_out) * terms * 1.01 + 2.0 ** -25).all())
    assert torch.all(dX[:, d_in:] == 7.0)
