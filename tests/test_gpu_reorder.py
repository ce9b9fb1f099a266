"""GPU parity of the locality reordering: permutation, relabelled CSR and row maps, called through
the C ABI, bit-exact against the reordering oracle; then the permutation-in / permutation-out
contract end to end (a layer on the relabelled graph, mapped back, against the forward oracle on
the original graph)."""
import numpy as np
import pytest
import torch

import synth
from oracle import ftc_oracle_reorder as OR
from parity import TOL, dev_graph, norm_err, quantise
from paper_2412_12218_amd import binding as B

pytestmark = pytest.mark.gpu

F32, F16, BF16 = torch.float32, torch.float16, torch.bfloat16


def say(msg):
    print(msg, flush=True)


def skewed_graph():
    """Degrees from 0 to 70 000 (a row longer than many sorting tiles), duplicates, unsorted
    columns, n not a multiple of anything convenient."""
    rng = np.random.default_rng(17)
    n = 9973
    deg = rng.integers(0, 40, size=n)
    deg[::7] = 0
    deg[100] = 70_000
    deg[101] = 4096
    deg[n - 1] = 2049
    row_ptr = np.zeros(n + 1, dtype=np.int32)
    row_ptr[1:] = np.cumsum(deg)
    col = rng.integers(0, n, size=int(row_ptr[-1])).astype(np.int32)
    return synth.Graph(n, row_ptr, col, "skewed")


@pytest.fixture(scope="module")
def graphs():
    return {
        "cfg1": synth.config_graph(1),
        "cfg2s": synth.config_graph(2, 0.2),
        "cfg5s": synth.config_graph(5, 1 / 32),
        "skewed": skewed_graph(),
        "one": synth.Graph(1, np.array([0, 1], dtype=np.int32), np.array([0], dtype=np.int32), "one"),
        "no_edges": synth.Graph(50, np.zeros(51, dtype=np.int32), np.zeros(0, dtype=np.int32), "no_edges"),
    }


@pytest.mark.parametrize("name", ["cfg1", "cfg2s", "cfg5s", "skewed", "one", "no_edges"])
@pytest.mark.parametrize("mode", [B.FTC_ORDER_DEGREE, B.FTC_ORDER_DEGREE_CLASSES])
def test_degree_order_and_permute_graph(graphs, name, mode):
    g = graphs[name]
    say(f"reorder {name} n={g.n} nnz={g.nnz} mode={mode}")
    perm_ref, inv_ref = OR.degree_order(g.row_ptr, mode)
    dg = dev_graph(g)
    perm, inv = B.ftc_degree_order(dg, mode)
    assert np.array_equal(perm.cpu().numpy().astype(np.int64), perm_ref)
    assert np.array_equal(inv.cpu().numpy().astype(np.int64), inv_ref)
    rp_ref, ci_ref = OR.permute_graph(g.row_ptr, g.col_idx, perm_ref, inv_ref)
    pg, flag = B.ftc_permute_graph(dg, perm, inv)
    assert int(flag.item()) == 0
    assert np.array_equal(pg.row_ptr.cpu().numpy().astype(np.int64), rp_ref)
    assert np.array_equal(pg.col_idx.cpu().numpy().astype(np.int64), ci_ref)
    pg2, _ = B.ftc_permute_graph(dg, perm, inv)                 # same answer again
    assert torch.equal(pg.col_idx, pg2.col_idx) and torch.equal(pg.row_ptr, pg2.row_ptr)


def test_permute_graph_with_a_callers_permutation(graphs):
    """Any permutation is accepted, not only the library's own orderings."""
    g = graphs["cfg2s"]
    rng = np.random.default_rng(4)
    perm_ref = rng.permutation(g.n)
    inv_ref = np.empty(g.n, dtype=np.int64)
    inv_ref[perm_ref] = np.arange(g.n)
    rp_ref, ci_ref = OR.permute_graph(g.row_ptr, g.col_idx, perm_ref, inv_ref)
    perm = torch.from_numpy(perm_ref.astype(np.int32)).cuda()
    inv = torch.from_numpy(inv_ref.astype(np.int32)).cuda()
    pg, flag = B.ftc_permute_graph(dev_graph(g), perm, inv)
    assert int(flag.item()) == 0
    assert np.array_equal(pg.row_ptr.cpu().numpy().astype(np.int64), rp_ref)
    assert np.array_equal(pg.col_idx.cpu().numpy().astype(np.int64), ci_ref)


def test_permute_graph_flags_what_is_not_a_permutation(graphs):
    g = graphs["cfg1"]
    dg = dev_graph(g)
    perm, inv = B.ftc_degree_order(dg)
    bad = perm.clone()
    bad[5] = bad[6]                                   # a repeated id
    _, flag = B.ftc_permute_graph(dg, bad, inv)
    assert int(flag.item()) == 1
    bad = perm.clone()
    bad[0] = g.n + 3                                  # out of range: must not be followed
    _, flag = B.ftc_permute_graph(dg, bad, inv)
    assert int(flag.item()) == 1
    bad_inv = inv.clone()
    bad_inv[9] = -1
    _, flag = B.ftc_permute_graph(dg, perm, bad_inv)
    assert int(flag.item()) == 1
    _, flag = B.ftc_permute_graph(dg, perm, inv)      # and the valid pair is still accepted
    assert int(flag.item()) == 0


@pytest.mark.parametrize("dtype,D,ld", [(F16, 32, 32), (F32, 16, 16), (BF16, 24, 24), (F16, 5, 5), (F32, 7, 12),
                                        (F16, 8, 24)])
def test_permute_rows(dtype, D, ld):
    n = 4099
    rng = np.random.default_rng(1)
    perm = rng.permutation(n)
    inv = np.empty(n, dtype=np.int64)
    inv[perm] = np.arange(n)
    full = torch.from_numpy(synth.normal_features(n, ld, seed=2)).to(dtype).cuda()
    X = full[:, :D]
    pd, idd = torch.from_numpy(perm.astype(np.int32)).cuda(), torch.from_numpy(inv.astype(np.int32)).cuda()
    Xp = B.ftc_permute_rows(X, pd)
    assert torch.equal(Xp.cpu(), X.cpu()[torch.from_numpy(perm)])
    back = B.ftc_permute_rows(Xp, idd)
    assert torch.equal(back, X.contiguous())
    bad = pd.clone()
    bad[3] = -7
    Xz = B.ftc_permute_rows(X, bad)
    assert torch.all(Xz[3] == 0) and torch.equal(Xz[4], Xp[4])


@pytest.mark.parametrize("name", ["cfg2s", "cfg5s", "skewed"])
def test_layers_on_the_relabelled_graph_match_the_original(oracle, graphs, name):
    """Permutation in, permutation out: GCN and AGNN layers computed on the relabelled graph and
    mapped back equal the oracle's layers on the original graph."""
    g = graphs[name]
    dg = dev_graph(g)
    perm, inv = B.ftc_degree_order(dg)
    pg, _ = B.ftc_permute_graph(dg, perm, inv)
    win = B.ftc_build_windows(pg)
    _, dinv = B.ftc_gcn_norm(pg, win, want_vals=False)
    Xd, X64 = quantise(synth.uniform_features(g.n, 64, seed=9), F16)
    Wd, W64 = quantise(synth.glorot_uniform(64, 16, seed=10), F16)
    out_p = B.ftc_gcn_layer(pg, win, None, B.ftc_permute_rows(Xd, perm), Wd, relu=True, dinv=dinv)
    out = B.ftc_permute_rows(out_p, inv)
    _, dinv64 = oracle.gcn_norm(g.row_ptr, g.col_idx)
    d32 = np.nan_to_num(dinv64, posinf=0.0).astype(np.float32).astype(np.float64)
    rows = np.repeat(np.arange(g.n), np.diff(g.row_ptr))
    ref, ab = oracle.gcn_layer(g.row_ptr, g.col_idx, d32[rows] * d32[g.col_idx], X64, W64, relu=True)
    err = norm_err(out, ref, ab)
    say(f"gcn layer through the reordering, {name}: err {err:.3e}")
    assert err < TOL[F16]
    Hd, H64 = quantise(synth.normal_features(g.n, 32, seed=11), F16)
    ref, ab, _ = oracle.agnn_layer(g.row_ptr, g.col_idx, H64, 1.0)
    out = B.ftc_permute_rows(B.ftc_agnn_layer(pg, win, B.ftc_permute_rows(Hd, perm)), inv)
    err = norm_err(out, ref, ab)
    say(f"agnn layer through the reordering, {name}: err {err:.3e}")
    assert err < TOL[F16]


@pytest.mark.parametrize("name", ["cfg1", "cfg5s", "skewed", "no_edges"])
def test_degree_stats_and_plan_from_device_numbers(graphs, name):
    """Sum of squared row lengths and longest row, exact; then the plan from the numbers the device
    produced (statistics + the window build's summary)."""
    g = graphs[name]
    deg = np.diff(g.row_ptr).astype(np.int64)
    dg = dev_graph(g)
    stats = B.ftc_degree_stats(dg).cpu().numpy()
    assert int(stats[0]) == int((deg * deg).sum()) and int(stats[1]) == int(deg.max())
    win = B.ftc_build_windows(dg)
    plan = B.ftc_plan_graph(g.n, g.nnz, int(stats[0]), int(win.summary[0].item()), 32, F16)
    say(f"plan {name}: {plan}")
    expect = name in ("cfg5s",) and g.n * 64 > 4 << 20
    assert (plan["reorder"] != B.FTC_ORDER_NONE) == expect
    if g.nnz:
        assert plan["reuse"] >= 1.0 and plan["skew"] >= 1.0 - 1e-9


# ------------------------------------------------------------------ the plan carried out
@pytest.mark.parametrize("which", ["rmat", "sbm", "small"])
def test_planned_graph_applies_the_plan_and_keeps_the_original_numbering(oracle, which):
    """PlannedGraph: statistics -> plan -> relabelled graph.  The skewed R-MAT graph is relabelled by degree
    class, the permuted block model gets the community trial and keeps it (its windows then share columns),
    a graph whose features fit one L2 is left alone; in every case a GCN layer and an AGNN layer run through
    enter() / leave() equal the oracle on the graph as given."""
    from paper_2412_12218_amd.models import PlannedGraph
    if which == "rmat":
        g, dtype, D, expect = synth.config_graph(5, 1 / 16), F16, 64, "degree classes"
    elif which == "sbm":
        g, dtype, D, expect = synth.config_graph(4, 0.05), BF16, 64, "communities"
    else:
        g, dtype, D, expect = synth.config_graph(1), F16, 32, "none"
    dg = dev_graph(g)
    pl = PlannedGraph(dg, D, dtype)
    say(f"planned {which}: n={g.n} nnz={g.nnz} plan={pl.plan} applied={pl.applied} sum_uniq {pl.sum_uniq_given} -> {pl.sum_uniq}")
    assert pl.applied == expect
    if which == "sbm":
        assert pl.sum_uniq < 0.98 * pl.sum_uniq_given
    _, dinv = B.ftc_gcn_norm(pl.g, pl.win, want_vals=False)
    Xd, X64 = quantise(synth.uniform_features(g.n, D, seed=9), dtype)
    Wd, W64 = quantise(synth.glorot_uniform(D, 16, seed=10), dtype)
    out = pl.leave(B.ftc_gcn_layer(pl.g, pl.win, None, pl.enter(Xd), Wd, relu=True, dinv=dinv))
    _, dinv64 = oracle.gcn_norm(g.row_ptr, g.col_idx)
    d32 = dinv64.astype(np.float32).astype(np.float64)
    rows = np.repeat(np.arange(g.n), np.diff(g.row_ptr))
    ref, ab = oracle.gcn_layer(g.row_ptr, g.col_idx, d32[rows] * d32[g.col_idx], X64, W64, relu=True)
    err = norm_err(out, ref, ab)
    say(f"  gcn layer on the planned graph: err {err:.3e}")
    assert err < TOL[dtype]
    Hd, H64 = quantise(synth.normal_features(g.n, D, seed=11), dtype)
    ref, ab, _ = oracle.agnn_layer(g.row_ptr, g.col_idx, H64, 1.0)
    out = pl.leave(B.ftc_agnn_layer(pl.g, pl.win, pl.enter(Hd)))
    err = norm_err(out, ref, ab)
    say(f"  agnn layer on the planned graph: err {err:.3e}")
    assert err < TOL[dtype]


def test_planned_graph_drops_a_community_trial_that_does_not_help():
    """The block model once more, this time already in community order (the graph the first plan produced):
    the plan proposes the trial again (the statistics cannot see the order), the relabelled windows share no
    more columns than before, and the graph stays as it is."""
    from paper_2412_12218_amd.models import PlannedGraph
    g = synth.config_graph(4, 0.05)
    first = PlannedGraph(dev_graph(g), 64, BF16)
    assert first.applied == "communities"
    pl = PlannedGraph(first.g, 64, BF16)
    say(f"planned twice: plan={pl.plan} applied={pl.applied} trial={getattr(pl, 'trial', None)}")
    assert pl.plan["reorder"] == B.FTC_ORDER_COMMUNITIES
    assert pl.applied == "none" and pl.trial["kept"] is False and pl.perm is None and pl.g is first.g


# ------------------------------------------------------------------ community ordering
def sbm_small():
    return synth.sbm(12, 200, 14 * 12 * 200, 2 * 12 * 200, seed=5)


@pytest.mark.parametrize("name", ["cfg1", "sbm", "skewed", "one", "no_edges"])
@pytest.mark.parametrize("rounds", [0, 1, 4])
def test_label_propagation(graphs, name, rounds):
    g = sbm_small() if name == "sbm" else graphs[name]
    say(f"label propagation {name} n={g.n} nnz={g.nnz} rounds={rounds}")
    ref = OR.label_propagation(g.row_ptr, g.col_idx, rounds)
    lab = B.ftc_label_propagation(dev_graph(g), rounds)
    assert np.array_equal(lab.cpu().numpy().astype(np.int64), ref)


def test_community_order_recovers_the_blocks_and_concentrates_the_columns(oracle):
    """Ten rounds on the permuted block model, then the ordering by label: bit-exact against the
    oracle, and the relabelled graph's windows hold far fewer distinct columns."""
    g = sbm_small()
    dg = dev_graph(g)
    lab = B.ftc_label_propagation(dg, 10)
    ref = OR.label_propagation(g.row_ptr, g.col_idx, 10)
    assert np.array_equal(lab.cpu().numpy().astype(np.int64), ref)
    perm, inv, flag = B.ftc_order_by_key(lab)
    perm_ref, inv_ref = OR.order_by_key(ref)
    assert int(flag.item()) == 0
    assert np.array_equal(perm.cpu().numpy().astype(np.int64), perm_ref)
    assert np.array_equal(inv.cpu().numpy().astype(np.int64), inv_ref)
    pg, pflag = B.ftc_permute_graph(dg, perm, inv)
    assert int(pflag.item()) == 0
    before = int(B.ftc_build_windows(dg).summary[0].item())
    after = int(B.ftc_build_windows(pg).summary[0].item())
    say(f"distinct window columns {before} -> {after} of {g.nnz} entries")
    assert after < 0.75 * before


def test_order_by_key_random_keys_and_negative_flag():
    rng = np.random.default_rng(3)
    n = 70_001
    keys = rng.integers(0, 50, size=n).astype(np.int32)
    keys[::1000] = rng.integers(1 << 20, (1 << 31) - 1, size=keys[::1000].size)     # all four digit passes matter
    perm_ref, inv_ref = OR.order_by_key(keys)
    perm, inv, flag = B.ftc_order_by_key(torch.from_numpy(keys).cuda())
    assert int(flag.item()) == 0
    assert np.array_equal(perm.cpu().numpy().astype(np.int64), perm_ref)
    assert np.array_equal(inv.cpu().numpy().astype(np.int64), inv_ref)
    keys[5] = -3
    _, _, flag = B.ftc_order_by_key(torch.from_numpy(keys).cuda())
    assert int(flag.item()) == 1


# ------------------------------------------------------------------ row-wise sorting: edges of the row classes
ROW_EDGES = [0, 1, 2, 31, 32, 33, 63, 64, 65, 255, 256, 257, 1023, 1024, 1025, 2048, 2049, 4096, 4097, 8191, 8192, 8193,
             16_384, 16_385, 32_768, 32_769, 40_000]


def edge_rows_graph(n, distinct, seed):
    """Rows of every length at which the row-wise kernels change, in random places; columns unsorted, with or
    without duplicates inside a row."""
    rng = np.random.default_rng(seed)
    deg = np.zeros(n, dtype=np.int64)
    at = rng.choice(n, size=3 * len(ROW_EDGES), replace=False)
    deg[at] = np.tile(ROW_EDGES, 3)
    deg[rng.choice(n, size=min(n, 3000), replace=False)] += rng.integers(0, 5, size=min(n, 3000))
    row_ptr = np.zeros(n + 1, dtype=np.int32)
    row_ptr[1:] = np.cumsum(deg)
    cols = []
    for i in np.nonzero(deg)[0]:
        cols.append(rng.choice(n, size=deg[i], replace=False) if distinct else rng.integers(0, max(1, n // 4), size=deg[i]))
    return synth.Graph(n, row_ptr, np.concatenate(cols).astype(np.int32), "edges")


def voted(rows, cand, n, keep):
    """Most frequent candidate per row, the smallest on a tie; rows without entries keep theirs."""
    key, votes = np.unique(rows * n + cand, return_counts=True)
    order = np.lexsort((-(key % n), votes, key // n))       # per row ascending: the last one wins
    r = (key // n)[order]
    last = np.r_[r[1:] != r[:-1], True]
    out = keep.copy()
    out[r[last]] = (key % n)[order][last]
    return out


@pytest.mark.parametrize("n", [65_537, 1 << 19, (1 << 19) + 1, (1 << 20) + 77, 1 << 22, (1 << 22) + 1])
@pytest.mark.parametrize("distinct", [True, False])
def test_row_lengths_at_the_edges_of_the_row_classes(n, distinct):
    """The last size is the first that sorts all entries at once instead of row by row; above 2^19 nodes longer rows are sorted
    in LDS."""
    g = edge_rows_graph(n, distinct, seed=n + distinct)
    say(f"row classes n={n} nnz={g.nnz} distinct={distinct}")
    rows = np.repeat(np.arange(n, dtype=np.int64), np.diff(g.row_ptr))
    col = g.col_idx.astype(np.int64)
    perm = np.random.default_rng(3).permutation(n)
    inv = np.empty(n, dtype=np.int64)
    inv[perm] = np.arange(n)
    dg = dev_graph(g)
    i32 = lambda a: torch.from_numpy(a.astype(np.int32)).cuda()
    pg, flag = B.ftc_permute_graph(dg, i32(perm), i32(inv))
    key = np.sort(inv[rows] * n + inv[col])
    assert int(flag.item()) == 0
    assert np.array_equal(pg.row_ptr.cpu().numpy(), np.r_[0, np.cumsum(np.diff(g.row_ptr)[perm])])
    assert np.array_equal(pg.col_idx.cpu().numpy(), key % n)
    label = np.arange(n, dtype=np.int64)
    for rounds in (1, 2):
        label = voted(rows, label[col], n, label)
        got = B.ftc_label_propagation(dg, rounds).cpu().numpy()
        assert np.array_equal(got, label), f"{rounds} rounds"


@pytest.mark.parametrize("kind,n,deg", [("blocks", 400_000, 34), ("uniform", 1_000_000, 16), ("skewed", 1 << 21, 8), ("directed", 1 << 20, 14),
                                        ("duplicates", 300_001, 45)])
def test_rounds_that_leave_out_the_rows_that_cannot_change(kind, n, deg):
    """12 M entries and more: rounds after the second one vote only on rows a column of which has changed.  Every number of rounds,
    against the same votes by sorting; columns that are unsorted, repeated, out of order with the rows that name them, hub rows;
    2^20 nodes are the last with a bit each."""
    gen = torch.Generator(device="cuda").manual_seed(n)
    m = n * deg
    if kind == "blocks":  # pairs inside communities of 200, shuffled: labels settle after some rounds
        perm = torch.randperm(n, generator=gen, device="cuda")
        c = torch.randint(n // 200, (m,), generator=gen, device="cuda") * 200
        r, c = (perm[c + torch.randint(200, (m,), generator=gen, device="cuda")] for _ in range(2))
    elif kind == "skewed":  # three quarters of the entries in a few rows of all classes
        hubs = torch.randint(3000, (m * 3 // 4,), generator=gen, device="cuda") ** 2 % 5000
        r = torch.cat([hubs, torch.randint(n, (m - m * 3 // 4,), generator=gen, device="cuda")])
        c = torch.randint(n, (m,), generator=gen, device="cuda") ** 2 % n
    else:
        r, c = (torch.randint(n, (m,), generator=gen, device="cuda") for _ in range(2))
        if kind == "duplicates":
            c = c // 50 * 50
        if kind == "directed":
            c = c * 3 // 4  # some nodes are nobody's column, and the pattern is not symmetric
    if kind == "uniform":
        r, c = torch.cat([r[:m // 2], c[:m // 2]]), torch.cat([c[:m // 2], r[:m // 2]])
    r, order = torch.sort(r, stable=True)
    c = c[order]
    row_ptr = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
    row_ptr[1:] = torch.cumsum(torch.bincount(r, minlength=n), 0)
    g = B.Graph(row_ptr, c.to(torch.int32))
    assert g.nnz >= 12_000_000
    label = torch.arange(n, device="cuda")
    for rounds in range(1, 12):
        key, votes = torch.unique(r * n + label[c], return_counts=True)
        best = torch.zeros(n, dtype=torch.int64, device="cuda").scatter_reduce_(0, key // n, votes * n + (n - 1 - key % n), "amax")
        label = torch.where(best > 0, n - 1 - best % n, label)
        assert torch.equal(B.ftc_label_propagation(g, rounds).long(), label), f"{rounds} rounds"


@pytest.mark.parametrize("n", [1, 511, 512, 513, (1 << 19) - 1, 1 << 19, (1 << 19) + 1, (1 << 22), (1 << 22) + 1])
def test_order_by_key_at_the_lines_of_its_tiles(n):
    """Keys of all four digits, many equal: stable, in a workspace of exactly the size that is asked for a graph without entries."""
    gen = torch.Generator(device="cuda").manual_seed(n)
    keys = torch.randint(1 << 31, (n,), generator=gen, device="cuda").to(torch.int32)
    keys[::3] = keys[::3] % 1000
    size = B.lib().ftc_reorder_workspace_bytes(n, 0)
    ws = torch.full((size + 4096,), 0x5a, dtype=torch.uint8, device="cuda")
    perm, inv, flag = B.ftc_order_by_key(keys, ws=ws[:size])
    ref = torch.sort(keys, stable=True).indices
    assert int(flag.item()) == 0 and torch.equal(perm.long(), ref)
    assert torch.equal(inv.long()[ref], torch.arange(n, device="cuda"))
    assert torch.all(ws[size:] == 0x5a)


@pytest.mark.parametrize("long_rows", [1, 200, 255, 256, 257, 1500])
@pytest.mark.parametrize("distinct", [True, False])
def test_few_and_many_rows_of_a_workgroup_each(long_rows, distinct):
    """Up to 256 rows of 1025 to 4096 entries those above 2048 are sorted by the kernel of the longer rows, from 257 on beside the short
    ones; with rows of every class around them."""
    rng = np.random.default_rng(long_rows)
    n = 9000
    deg = rng.integers(0, 40, size=n)
    at = rng.choice(n, size=long_rows + 120, replace=False)
    deg[at[:long_rows]] = np.resize([4096, 1025, 2049, 2048, 3000], long_rows)
    deg[at[long_rows:]] = np.resize([65, 128, 129, 256, 257, 512, 513, 1024, 4097, 8192, 8193], 120)
    row_ptr = np.zeros(n + 1, dtype=np.int32)
    row_ptr[1:] = np.cumsum(deg)
    rows = np.repeat(np.arange(n, dtype=np.int64), deg)
    col = np.concatenate([rng.choice(n, size=d, replace=False) if distinct else rng.integers(0, n // 4, size=d) for d in deg]).astype(np.int64)
    perm = rng.permutation(n)
    inv = np.empty(n, dtype=np.int64)
    inv[perm] = np.arange(n)
    dg = dev_graph(synth.Graph(n, row_ptr, col.astype(np.int32), "long rows"))
    i32 = lambda a: torch.from_numpy(a.astype(np.int32)).cuda()
    pg, flag = B.ftc_permute_graph(dg, i32(perm), i32(inv))
    assert int(flag.item()) == 0
    assert np.array_equal(pg.col_idx.cpu().numpy(), np.sort(inv[rows] * n + inv[col]) % n)
    label = np.arange(n, dtype=np.int64)
    for rounds in (1, 2, 3):
        label = voted(rows, label[col], n, label)
        assert np.array_equal(B.ftc_label_propagation(dg, rounds).cpu().numpy(), label), f"{rounds} rounds"
