"""Window build by a wave per window (at most 1024 edges, two-level bitmap): window sizes at the edges of its steps and queues, column
counts on both sides of its lines, any order of columns, repeated ones; against sorted distinct (window, column) pairs, exactly."""
import pytest
import torch

from paper_2412_12218_amd import binding as B

pytestmark = pytest.mark.gpu
SIZES = [0, 1, 2, 63, 64, 65, 255, 256, 257, 511, 512, 513, 767, 768, 1023, 1024, 1025, 2047, 2048, 2049, 4095, 4096, 4097, 9000, 33_000]


def exact(row_ptr, cols, n, blk_h):
    row_ptr, cols = row_ptr.long(), cols.long()
    rows = torch.repeat_interleave(torch.arange(n, device="cuda"), row_ptr[1:] - row_ptr[:-1])
    n_win = (n + blk_h - 1) // blk_h
    pairs, where = torch.unique((rows // blk_h) * n + cols, return_inverse=True)
    counts = torch.bincount(pairs // n, minlength=n_win)
    start = torch.zeros(n_win + 1, dtype=torch.int64, device="cuda")
    start[1:] = torch.cumsum(counts, 0)
    return rows, where - start[rows // blk_h], (counts + 7) // 8, start, pairs % n


def check(row_ptr, cols, n, blk_h, side):
    g = B.Graph(row_ptr, cols)
    w = B.ftc_build_windows_concurrent(g, B.SideStreams() if side else None, blk_h=blk_h)
    e2r, e2c, blocks, start, uniq = exact(row_ptr, cols, n, blk_h)
    assert torch.equal(w.win_col_ptr.long(), start) and torch.equal(w.block_partition.long(), blocks)
    assert w.summary.tolist() == [uniq.numel(), int(blocks.sum())]
    assert torch.equal(w.edge_to_row.long(), e2r) and torch.equal(w.edge_to_col.long(), e2c)
    assert torch.equal(w.win_cols[:uniq.numel()].long(), uniq)


def window_sizes_graph(n, blk_h, fill, seed):
    """Windows of every size in SIZES, three times, in random places; the others hold `fill` entries.  Rows of a window share its
    entries unevenly; columns in any order: spread over all, packed into a few words, one column only, the ends of the range."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    n_win = (n + blk_h - 1) // blk_h
    size = torch.full((n_win,), fill, dtype=torch.int64, device="cuda")
    at = torch.randperm(n_win - 1, generator=gen, device="cuda")[:3 * len(SIZES)]
    size[at] = torch.tensor(SIZES * 3, device="cuda")
    win = torch.repeat_interleave(torch.arange(n_win, device="cuda"), size)
    m = win.numel()
    in_win = torch.minimum(torch.rand(m, generator=gen, device="cuda"), torch.rand(m, generator=gen, device="cuda")) * blk_h
    rows = torch.minimum(win * blk_h + in_win.long().clamp(max=blk_h - 1), torch.full_like(win, n - 1))
    rows = torch.sort(rows).values
    kind = win % 4
    spread = torch.randint(n, (m,), generator=gen, device="cuda")
    packed = (win * 977 % n + torch.randint(100, (m,), generator=gen, device="cuda")) % n
    ends = torch.where(torch.rand(m, generator=gen, device="cuda") < 0.5, spread % 70, n - 1 - spread % 70)
    cols = torch.where(kind == 0, packed, torch.where(kind == 1, torch.where(win % 3 == 0, win % n, ends), spread))
    row_ptr = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
    row_ptr[1:] = torch.cumsum(torch.bincount(rows, minlength=n), 0)
    return row_ptr, cols.to(torch.int32)


@pytest.mark.parametrize("n,blk_h,fill", [(65_537, 16, 100), (131_072, 16, 127), (131_072, 16, 129), (131_072, 16, 5), (65_537, 16, 60), (80_000, 16, 150), (100_000, 64, 40), (131_073, 16, 40), (200_003, 16, 300),
                                          (200_003, 32, 639), (262_144, 16, 600), (262_144, 64, 500), (262_144, 8, 20), (262_145, 16, 300),
                                          (262_145, 64, 700), (500_001, 16, 10), (1 << 20, 16, 260), ((1 << 20) + 1, 16, 260)])
@pytest.mark.parametrize("side", [False, True])
def test_window_sizes(n, blk_h, fill, side):
    check(*window_sizes_graph(n, blk_h, fill, seed=n + fill), n, blk_h, side)
