"""The edge-balanced kernels where a range of entries can go wrong: rows that end at, before and behind the ends of runs and
ranges, rows without entries among them, more rows than a range has marks for, a last range of one entry, long and short ranges,
lanes beyond the row, and feature matrices of more than 4 GiB.  Compared with plain fp64 torch, element by element,
relative to the sum of the absolute terms; 1e-5, the bar of fp32 sums, also for 16-bit inputs (they are taken as they are)."""
import numpy as np
import pytest
import torch

from paper_2412_12218_amd import binding as B

pytestmark = pytest.mark.gpu
F32, F16, BF16 = torch.float32, torch.float16, torch.bfloat16


def row_lengths(which):
    if which == "edges":  # around the lengths of runs (8 to 128) and ranges (128, 512)
        return [0, 0, 1, 7, 8, 9, 0, 31, 32, 33, 1, 127, 128, 129, 0, 0, 3, 511, 512, 513, 1, 1, 255, 256, 257, 64, 0, 1025, 2, 1, 5000, 6]
    if which == "ones":  # more row starts than half a range
        return [1] * 700 + [0] * 50 + [1, 2] * 300 + [1]
    if which == "aligned":  # every row ends with a range
        return [128] * 8 + [512] * 4 + [64, 64] * 4
    return [3000] + [0] * 600 + [1] * 3  # one row over many ranges, then a gap of rows without entries


def graph(lengths, seed=0):
    rng = np.random.default_rng(seed)
    n = len(lengths)
    ptr = np.zeros(n + 1, dtype=np.int32)
    ptr[1:] = np.cumsum(lengths)
    return B.Graph.from_numpy(ptr, rng.integers(0, n, size=int(ptr[-1])).astype(np.int32))


def rows_of(g):
    rp = g.row_ptr.long()
    return torch.repeat_interleave(torch.arange(g.n, device="cuda"), rp[1:] - rp[:-1])


def close(got, ref, terms, tol=1e-5):
    err = (got.double() - ref).abs() / terms.clamp(min=1e-300)
    assert torch.all(got[terms == 0] == 0)
    assert float(torch.where(terms > 0, err, torch.zeros_like(err)).max()) <= tol


def check_spmm(g, win, vals, X, out):
    rows, cols = rows_of(g), g.col_idx.long()
    t = X.double()[cols] * (1.0 if vals is None else vals.double()[:, None])
    ref = torch.zeros(out.shape, dtype=torch.float64, device="cuda")
    close(out, ref.clone().index_add_(0, rows, t), ref.clone().index_add_(0, rows, t.abs()))


def attention(g, X, beta):
    rows, cols = rows_of(g), g.col_idx.long()
    H = X.double()
    Hn = H / H.norm(dim=1).clamp(min=1e-12)[:, None]
    w = torch.exp(beta * (Hn[rows] * Hn[cols]).sum(1) - abs(beta))
    z = torch.zeros(g.n, dtype=torch.float64, device="cuda").index_add_(0, rows, w)
    p = w / z[rows]
    t = H[cols] * p[:, None]
    ref = torch.zeros(X.shape, dtype=torch.float64, device="cuda")
    return p, z, ref.clone().index_add_(0, rows, t), ref.clone().index_add_(0, rows, t.abs())


def smallest_workspace(call, nbytes):
    """The smallest workspace (a multiple of 256 bytes) that a call accepts: with it the kernels use their longest ranges."""
    lo, hi = 0, nbytes // 256 + 1
    while hi - lo > 1:
        mid = (lo + hi) // 2
        try:
            call(torch.empty(mid * 256, dtype=torch.uint8, device="cuda"))
            hi = mid
        except B.FtcError:
            lo = mid
    return torch.full((hi * 256,), 0xff, dtype=torch.uint8, device="cuda")


SHAPES = [(F16, 32), (F16, 64), (BF16, 128), (F16, 40), (BF16, 24), (F32, 128), (F32, 32), (F32, 12), (F16, 16), (F16, 8), (F16, 256)]


@pytest.mark.parametrize("which,times", [("edges", 1), ("ones", 1), ("aligned", 1), ("gap", 1), ("edges", 60), ("ones", 330), ("aligned", 150)])
@pytest.mark.parametrize("dtype,D", SHAPES)
def test_rows_at_the_ends_of_runs_and_ranges(which, times, dtype, D):
    """Once: the kernels for small graphs, which have one launch and cut no rows (a mean row of at most 64 entries is theirs); many times
    over, more than half a million entries: the edge-balanced ones."""
    lengths = row_lengths(which) * times
    g = graph(lengths + [0] * (sum(lengths) // 64 if times == 1 else 0))
    assert times == 1 or g.nnz > 512 << 10
    win = B.ftc_build_windows(g)
    gen = torch.Generator(device="cuda").manual_seed(D)
    X = torch.randn((g.n, D), generator=gen, device="cuda").to(dtype)
    vals = torch.rand(g.nnz, generator=gen, device="cuda") + 0.5
    L = B.lib()
    long_ws = smallest_workspace(lambda ws: B.ftc_spmm(g, win, vals, X, ws=ws), L.ftc_spmm_workspace_bytes(g.n, g.nnz, D))
    for ws in (None, long_ws):
        for v in (vals, None):
            check_spmm(g, win, v, X, B.ftc_spmm(g, win, v, X, ws=ws))
    p, z, ref, terms = attention(g, X, 1.5)
    nbytes = L.ftc_agnn_layer_workspace_bytes(g.n, g.nnz, D)
    long_ws = smallest_workspace(lambda ws: B.ftc_agnn_layer(g, win, X, beta=1.5, ws=ws), nbytes)
    for ws in (None, long_ws):
        close(B.ftc_agnn_layer(g, win, X, beta=1.5, ws=ws), ref, terms)
        row_z = torch.empty(g.n, device="cuda")
        out32 = torch.empty((g.n, (D + 3) // 4 * 4), device="cuda")
        close(B.ftc_agnn_layer(g, win, X, beta=1.5, row_z=row_z, out_f32=out32, ws=ws), ref, terms)
        close(out32[:, :D], ref, terms)
        close(row_z, z, z)
        edge_p = torch.empty(g.nnz, device="cuda")
        close(B.ftc_agnn_layer(g, win, X, beta=1.5, edge_p=edge_p, ws=ws), ref, terms)
        close(edge_p, p, p)


@pytest.mark.parametrize("dtype,D", [(F16, 8), (BF16, 5), (F32, 3), (F16, 16), (BF16, 12), (F32, 8), (F32, 6)])
@pytest.mark.parametrize("times", [60, 240])
def test_output_scales_of_narrow_rows(dtype, D, times):
    """Rows of at most 32 bytes: their scales are staged where a range of entries has at most 128 rows; more, up to 128 and one row in a
    range, long rows over many; 4 and 16 entries a lane."""
    g = graph(([1] * 700 + [5] * 300 + [8] * 128 + [1024, 3, 0, 0, 2000, 17] + [40] * 30 + [3000]) * times)
    assert g.nnz > (512 << 10 if times == 60 else 2 << 20)
    win = B.ftc_build_windows(g)
    gen = torch.Generator(device="cuda").manual_seed(D)
    ld = (D + 7) // 8 * 8
    X = torch.randn((g.n, ld), generator=gen, device="cuda").to(dtype)[:, :D]
    vals, scale = torch.rand(g.nnz, generator=gen, device="cuda") + 0.5, torch.rand(g.n, generator=gen, device="cuda") + 0.5
    rows, cols, s = rows_of(g), g.col_idx.long(), scale.double()[:, None]
    for v in (vals, None):
        t = X.double()[cols] * (1.0 if v is None else v.double()[:, None])
        zero = torch.zeros((g.n, D), dtype=torch.float64, device="cuda")
        ref, terms = zero.clone().index_add_(0, rows, t) * s, zero.clone().index_add_(0, rows, t.abs()) * s
        for relu in (False, True):
            out = torch.full((g.n, ld), 7.0, device="cuda")
            B.ftc_spmm(g, win, v, X, out=out[:, :D], out_scale=scale, relu=relu)
            close(out[:, :D], torch.relu(ref) if relu else ref, terms)
            assert torch.all(out[:, D:] == 7.0)


@pytest.mark.parametrize("dtype,D", [(F16, 32), (F32, 32), (F16, 16), (F32, 4)])
def test_feature_matrix_of_more_than_4_gib(dtype, D):
    n, ld = 70_000, 32_768 if dtype == F16 else 16_384  # 4.6 GB, most of it between the rows
    rng = np.random.default_rng(1)
    lengths = rng.integers(1, 8, size=n)
    lengths[5] = 3000
    g = graph(list(lengths))
    win = B.ftc_build_windows(g)
    X = torch.empty((n, ld), dtype=dtype, device="cuda")[:, :D]
    X.copy_(torch.randn((n, D), device="cuda"))
    vals = torch.rand(g.nnz, device="cuda") + 0.5
    check_spmm(g, win, vals, X, B.ftc_spmm(g, win, vals, X))
    if D >= 32:
        _, _, ref, terms = attention(g, X, 1.5)
        close(B.ftc_agnn_layer(g, win, X, beta=1.5), ref, terms)


def symmetric_graph(n, rng):
    """Rows of all kinds: two hubs, a ring, pairs far apart, every tenth node without entries."""
    u = [np.arange(1, n), np.full(n // 2, 3), np.full(n - 5, n - 2), rng.integers(0, n, 3 * n)]
    v = [np.arange(n - 1), np.arange(n // 2), np.arange(n - 5), rng.integers(0, n, 3 * n)]
    u, v = np.concatenate(u), np.concatenate(v)
    keep = (u % 10 != 7) & (v % 10 != 7)
    u, v = u[keep], v[keep]
    key = np.unique(np.concatenate([u * n + v, v * n + u]))
    ptr = np.zeros(n + 1, dtype=np.int32)
    ptr[1:] = np.cumsum(np.bincount(key // n, minlength=n))
    return ptr, (key % n).astype(np.int32)


def attention_gradients(g, X, beta, dY):
    X = X.double().clone().requires_grad_()
    b = torch.tensor(float(beta), dtype=torch.float64, device="cuda", requires_grad=True)
    rows, cols = rows_of(g), g.col_idx.long()
    Xn = X / X.norm(dim=1).clamp(min=1e-12)[:, None]
    w = torch.exp(b * (Xn[rows] * Xn[cols]).sum(1))
    z = torch.zeros(g.n, dtype=torch.float64, device="cuda").index_add(0, rows, w)
    out = torch.zeros(X.shape, dtype=torch.float64, device="cuda").index_add(0, rows, X[cols] * (w / z[rows])[:, None])
    out.backward(dY.double())
    return X.grad, b.grad


def dbeta_bar(g, X, beta, dY):
    """What the roundings of dbeta's terms ds_e c_e add up to: about twenty of 2^-24 in each, independent of one another; four standard
    deviations."""
    p, _, Y, _ = attention(g, X, beta)
    rows, cols = rows_of(g), g.col_idx.long()
    H, d = X.double(), dY.double()
    Hn = H / H.norm(dim=1).clamp(min=1e-12)[:, None]
    ds = p * ((d[rows] * H[cols]).sum(1) - (d * Y).sum(1)[rows])
    return 4 * 20 * 2.0 ** -24 * float((ds * (Hn[rows] * Hn[cols]).sum(1)).norm())


@pytest.mark.parametrize("dtype,D,pad", [(F16, 32, 0), (F16, 64, 0), (BF16, 40, 0), (F32, 32, 0), (F32, 128, 0), (F16, 16, 0), (F32, 12, 0),
                                         (F16, 32, 3), (F32, 128, 1), (BF16, 128, 0), (F32, 3, 5), (F32, 6, 2), (F16, 6, 2)])
def test_single_pass_backward_writes_complete_gradients(dtype, D, pad):
    n = 2003
    ptr, cols = symmetric_graph(n, np.random.default_rng(D))
    g = B.Graph.from_numpy(ptr, cols)
    win = B.ftc_build_windows(g)
    gen = torch.Generator(device="cuda").manual_seed(D)
    ld = D if D >= 8 else 8  # 16-byte aligned rows
    X = torch.randn((n, ld), generator=gen, device="cuda").to(dtype)[:, :D]
    dY = torch.randn((n, ld), generator=gen, device="cuda").to(dtype)[:, :D]
    X[11] *= 1e-4
    z = torch.empty(n, device="cuda")
    y32 = torch.empty((n, (D + 3) // 4 * 4), device="cuda")
    B.ftc_agnn_layer(g, win, X, beta=1.5, out=torch.empty((n, ld), device="cuda")[:, :D], row_z=z, out_f32=y32)
    ref, dbeta = attention_gradients(g, X, 1.5, dY)
    buf = torch.full((n, D + pad), 7.0, device="cuda")  # with padding: rows that are not 16-byte aligned
    dH, db = B.ftc_agnn_layer_backward_fused(g, win, X, z, y32[:, :D], dY, beta=1.5, dH=buf[:, :D])
    assert torch.all(buf[:, D:] == 7.0)
    empty = g.row_ptr[1:] == g.row_ptr[:-1]
    assert int(empty.sum()) > 100 and torch.all(dH[empty] == 0)
    # fp32 sums: relative to the largest element of the row (at least 1, the size of dY)
    scale = ref.abs().max(dim=1).values.clamp(min=1.0)
    assert float(((dH.double() - ref).abs().max(dim=1).values / scale).max()) <= 1e-5
    bar = dbeta_bar(g, X, 1.5, dY)
    print(f"dbeta {float(db):.6f}, error {abs(float(db) - float(dbeta)):.2e}, bar {bar:.2e}", flush=True)
    assert abs(float(db) - float(dbeta)) <= bar


def ring(n, hops):
    """Every node with its 2 * hops neighbours at the given distances: a symmetric pattern, ascending rows."""
    rng = np.random.default_rng(hops)
    d = rng.choice(np.arange(1, n // 2), size=hops, replace=False)
    cols = np.sort((np.arange(n)[:, None] + np.concatenate([d, n - d])[None]) % n, axis=1)
    return B.Graph.from_numpy((np.arange(n + 1) * 2 * hops).astype(np.int32), cols.reshape(-1).astype(np.int32))


@pytest.mark.parametrize("features", ["signed", "behind a ReLU"])
@pytest.mark.parametrize("beta", [1.0, -1.0, 3.0, 1e-6])
@pytest.mark.parametrize("ydt", [F32, F16, BF16])
@pytest.mark.parametrize("dtype,D,hops", [(F32, 32, 32), (F16, 32, 16), (F32, 128, 32)])
def test_dbeta_is_as_exact_as_the_plain_sum(dtype, D, hops, ydt, beta, features):
    """dbeta = sum of ds_e c_e.  What a rounded Y puts t_i = <dY_i, Y_i> off by, d_i, enters with what is left of the row's mean
    cosine c_i: no more than four standard deviations of independent errors d_i c_i, the plain sum's, and the roundings of the
    entries in fp32 (of about twenty operations each, 2^-24 every one, independent of one another)."""
    n = 2003
    g = ring(n, hops)
    gen = torch.Generator(device="cuda").manual_seed(D + hops)
    H = torch.randn((n, D), generator=gen, device="cuda")
    H = (torch.relu(H) if features != "signed" else H).to(dtype)
    dY = torch.randn((n, D), generator=gen, device="cuda").to(dtype)
    rows, cols = rows_of(g), g.col_idx.long()
    p, z, Y, _ = attention(g, H, beta)
    Hn = H.double() / H.double().norm(dim=1, keepdim=True)
    c = (Hn[rows] * Hn[cols]).sum(1)
    t = (dY.double() * Y).sum(1)
    ds = p * ((dY.double()[rows] * H.double()[cols]).sum(1) - t[rows])
    Yq = Y.to(ydt)
    off = (dY.double() * Yq.double()).sum(1) - t
    mean = torch.zeros(n, dtype=torch.float64, device="cuda").index_add_(0, rows, p * c)
    bar = 4 * float((off * mean).norm()) + 20 * 2.0 ** -24 * 4 * float((ds * c).norm())
    win = B.ftc_build_windows(g)
    _, db = B.ftc_agnn_layer_backward_fused(g, win, H, z.float(), Yq, dY, beta=beta)
    err = abs(float(db) - float((ds * c).sum()))
    print(f"dbeta {dtype} D={D} {2 * hops} neighbours Y {ydt} beta {beta} {features}: error {err:.2e}, bar {bar:.2e}", flush=True)
    assert err <= bar


def test_single_pass_backward_of_more_than_4_gib():
    """Copies of one graph side by side, 4.3 M nodes with rows of 1 KiB in the workspace: every copy has the gradients of the one."""
    n, copies, D = 43_000, 100, 128
    ptr, cols = symmetric_graph(n, np.random.default_rng(3))
    nnz = int(ptr[-1])
    small = B.Graph.from_numpy(ptr, cols)
    k = torch.arange(copies, device="cuda", dtype=torch.int32)[:, None]
    row_ptr = torch.cat([(small.row_ptr[None, :-1] + k * nnz).reshape(-1), torch.tensor([copies * nnz], dtype=torch.int32, device="cuda")])
    big = B.Graph(row_ptr, (small.col_idx[None] + k * n).reshape(-1).contiguous())
    gen = torch.Generator(device="cuda").manual_seed(0)
    X, dY = (torch.randn((n, D), generator=gen, device="cuda") for _ in range(2))
    results = []
    for g, rep in ((small, 1), (big, copies)):
        win = B.ftc_build_windows(g)
        H, d = X.repeat(rep, 1), dY.repeat(rep, 1)
        z = torch.empty(g.n, device="cuda")
        Y = B.ftc_agnn_layer(g, win, H, beta=1.0, row_z=z)
        results.append(B.ftc_agnn_layer_backward_fused(g, win, H, z, Y, d, beta=1.0))
    (a, da), (b, db) = results
    assert float((b.view(copies, n, D) - a).abs().max()) <= 1e-5 * float(a.abs().max())
    bar = dbeta_bar(small, X, 1.0, dY)
    print(f"dbeta {float(da):.6f}, of a copy {float(db) / copies:.6f}, bar {bar:.2e}", flush=True)
    assert abs(float(db) / copies - float(da)) <= 2 * bar
