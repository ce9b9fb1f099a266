"""Workloads by which the framework's speed is followed: what its users have it do, through its public entry points.

A case is a dict of plain values.  listed() names the standing ones, draw() makes more of the same ranges,
prepare() makes what a program has in hand before the call, run() is one pass, work() what a pass cannot do
without, tolerance() how far two correct implementations may be apart, exact() the same in 64 bits in plain torch.

Graphs are those of the benchmark configurations, made on the GPU: uniform random ("uniform"), power law
("powerlaw"), block model ("blocks") and R-MAT ("rmat"); undirected, without duplicates, with self-loops, columns
ascending inside a row.
"""
import math

import torch

from paper_2412_12218_amd import binding as B
from paper_2412_12218_amd.models import HotPath, PlannedGraph, TrainPath

DTYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
SIZE = {"f32": 4, "f16": 2, "bf16": 2}
BETAS = [1.0, 0.9, 1.1, 1.0]  # propagation weights of the AGNN layers (learnable, they start at 1)


def listed():
    return [
        # One aggregation on the smallest graph (2048 nodes, average degree 8, fp32, 16 columns): a call that
        # is all latency, as in a serving loop over small graphs.
        dict(name="small_spmm", kind="spmm", graph="uniform", n=2048, deg=8, d=16, dtype="f32"),
        # A whole forward pass (graph transformation, 2-layer GCN, 4-layer AGNN) on a graph the size of the
        # citation networks: few nodes, 1433 features in unpadded rows, 7 classes.
        dict(name="citation_step", kind="step", graph="uniform", n=2708, deg=4, d_in=1433, gcn=16, agnn=32, n_out=7,
             dtype="f16"),
        # The graph transformation alone, on the power-law graph with 200 000 nodes: what a program pays
        # when its graph changes.
        dict(name="powerlaw_windows", kind="windows", graph="powerlaw", n=200_000, deg=20),
        # One GCN layer, 100 000 nodes, power law, fp16 128 -> 32.
        dict(name="powerlaw_gcn_layer", kind="gcn_layer", graph="powerlaw", n=100_000, deg=16, d_in=128, d_out=32,
             dtype="f16"),
        # One AGNN layer that also returns its attention weights (scores, edge softmax and aggregation as
        # separate steps), 200 000 nodes, power law, fp16, 32 columns.
        dict(name="powerlaw_attention", kind="attention", graph="powerlaw", n=200_000, deg=20, d=32, beta=1.0,
             dtype="f16"),
        # The large aggregation with edge values: block model with a million nodes, bf16, 64 columns.
        dict(name="blocks_spmm", kind="spmm", graph="blocks", n=1_000_000, deg=32, d=64, dtype="bf16"),
        # The dense update of a first layer on many input features in fp32: unpadded odd rows.
        dict(name="wide_update", kind="update", n=100_000, d_in=1433, d_out=16, dtype="f32"),
        # Forward and backward of the 2-layer GCN in fp32: 300 features, hidden size 128, 10 classes.
        dict(name="gcn_train", kind="gcn_train", graph="powerlaw", n=100_000, deg=16, d_in=300, gcn=128, n_out=10,
             dtype="f32"),
        # Forward and backward of the AGNN model with 16-bit activations on the million-node R-MAT graph.
        dict(name="rmat_agnn_train", kind="agnn_train", graph="rmat", n=1 << 20, deg=32, d_in=128, agnn=32, n_out=8,
             dtype="f16"),
        # The benchmark's step: the whole forward pass on the million-node R-MAT graph.
        dict(name="rmat_step", kind="step", graph="rmat", n=1 << 20, deg=32, d_in=128, gcn=16, agnn=32, n_out=8,
             dtype="f16"),
        # Preparation of a graph before long use: statistics, plan and relabelling by degree class ...
        dict(name="rmat_plan", kind="plan", graph="rmat", n=1 << 20, deg=32, d=32, dtype="f16"),
        # ... and the trial of the community ordering, for a graph with flat degrees.
        dict(name="blocks_plan", kind="plan", graph="blocks", n=1_000_000, deg=32, d=64, dtype="bf16"),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_graph(rng, lo, hi):
    kind = rng.choice(["uniform", "powerlaw", "blocks", "rmat"])
    n = _log_uniform(rng, lo, hi)
    deg = rng.choice([4, 8, 16, 20, 32])
    if kind == "rmat":
        n = 1 << int(round(math.log2(n)))
    elif kind == "blocks":
        n = max(2, n // 1000) * 1000
    return dict(graph=kind, n=n, deg=deg)


def draw(rng):
    kind = rng.choice(["spmm", "step", "windows", "gcn_layer", "attention", "update", "gcn_train", "agnn_train", "plan"])
    dtype = rng.choice(["f32", "f16", "bf16"])
    classes = rng.choice([2, 3, 6, 7, 8, 10, 16, 22, 40, 47, 64])
    if kind == "spmm":
        return dict(kind=kind, **_draw_graph(rng, 1000, 500_000), d=rng.choice([6, 7, 8, 10, 16, 22, 32, 40, 47, 64, 96, 128]),
                    dtype=dtype)
    if kind == "step":
        return dict(kind=kind, **_draw_graph(rng, 1000, 300_000), d_in=_log_uniform(rng, 16, 512), gcn=rng.choice([8, 16, 32, 64]),
                    agnn=rng.choice([8, 16, 24, 32, 64]), n_out=classes, dtype=dtype)
    if kind == "windows":
        return dict(kind=kind, **_draw_graph(rng, 1000, 1_000_000))
    if kind == "gcn_layer":
        return dict(kind=kind, **_draw_graph(rng, 1000, 300_000), d_in=_log_uniform(rng, 16, 1024),
                    d_out=rng.choice([16, 32, 64, 128, classes]), dtype=dtype)
    if kind == "attention":
        return dict(kind=kind, **_draw_graph(rng, 1000, 500_000), d=rng.choice([8, 16, 32, 40, 64, 128]),
                    beta=round(rng.uniform(0.5, 4.0), 2), dtype=dtype)
    if kind == "update":
        n = _log_uniform(rng, 1000, 400_000)
        return dict(kind=kind, n=n, d_in=_log_uniform(rng, 16, min(4000, 150_000_000 // n)),
                    d_out=rng.choice([16, 32, 64, 128, classes]), dtype=dtype)
    if kind == "gcn_train":
        return dict(kind=kind, **_draw_graph(rng, 1000, 200_000), d_in=_log_uniform(rng, 16, 512), gcn=rng.choice([16, 32, 64, 128]),
                    n_out=classes, dtype=dtype)
    if kind == "agnn_train":
        return dict(kind=kind, **_draw_graph(rng, 1000, 200_000), d_in=_log_uniform(rng, 16, 512), agnn=rng.choice([16, 32, 64]),
                    n_out=classes, dtype=dtype)
    return dict(kind=kind, **_draw_graph(rng, 70_000, 500_000), d=rng.choice([32, 64, 128]), dtype=dtype)


# ---- inputs -------------------------------------------------------------------------------------------
def _generator(seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed * 1_000_003 + 17)
    return gen


def _pair_count(case):
    """Distinct undirected pairs of a graph: what sampling n * deg / 2 pairs leaves without loops and duplicates, about."""
    kept = {"uniform": 0.99, "powerlaw": 0.9, "blocks": 0.98, "rmat": 0.93}[case["graph"]]
    n = case["n"]
    return int(min(n * case["deg"] // 2 * kept, n * (n - 1) // 8))


def _entries(case):
    """Stored entries: both directions of every pair, and the self-loops."""
    return 2 * _pair_count(case) + case["n"]


def _sampler(case, gen):
    """sample(m): the endpoints of m undirected pairs, loops and duplicates among them."""
    n, deg = case["n"], case["deg"]
    ints = lambda hi, k: torch.randint(hi, (k,), generator=gen, device="cuda")
    if case["graph"] == "uniform":
        return lambda m: (ints(n, m), ints(n, m))
    if case["graph"] == "powerlaw":  # weights (i + i0)^(-1/(gamma - 1)), the largest sqrt(deg * n), numbering shuffled
        alpha = 1.0 / (2.2 - 1.0)
        i = torch.arange(n, device="cuda", dtype=torch.float64)
        lo, hi = 1e-6, float(n)
        for _ in range(40):
            mid = 0.5 * (lo + hi)
            w = (i + mid) ** -alpha
            if deg * n * float(w[0] / w.sum()) > math.sqrt(deg * n):
                lo = mid
            else:
                hi = mid
        cdf = torch.cumsum((i + hi) ** -alpha, 0)
        cdf = cdf / cdf[-1]
        perm = torch.randperm(n, generator=gen, device="cuda")
        rand = lambda k: torch.rand(k, generator=gen, device="cuda", dtype=torch.float64)
        pick = lambda m: perm[torch.searchsorted(cdf, rand(m)).clamp_(max=n - 1)]
        return lambda m: (pick(m), pick(m))
    if case["graph"] == "blocks":  # communities of 1000 nodes, 7 of 8 pairs inside one, numbering shuffled
        perm = torch.randperm(n, generator=gen, device="cuda")

        def blocks(m):
            inside = m * 7 // 8
            c = ints(n // 1000, inside) * 1000
            u = torch.cat([c + ints(1000, inside), ints(n, m - inside)])
            v = torch.cat([c + ints(1000, inside), ints(n, m - inside)])
            return perm[u], perm[v]
        return blocks

    def rmat(m):  # quadrants 0.57, 0.19, 0.19, 0.05
        u = torch.zeros(m, dtype=torch.int64, device="cuda")
        v = torch.zeros(m, dtype=torch.int64, device="cuda")
        for _ in range(n.bit_length() - 1):
            r = torch.rand(m, generator=gen, device="cuda")
            u = 2 * u + (r >= 0.76)
            v = 2 * v + (((r >= 0.57) & (r < 0.76)) | (r >= 0.95))
        return u, v
    return rmat


def _csr(case, gen):
    """Exactly _pair_count(case) distinct pairs, as a CSR adjacency: the sizes depend on the case alone."""
    n, want = case["n"], _pair_count(case)
    sample = _sampler(case, gen)
    pairs = torch.empty(0, dtype=torch.int64, device="cuda")
    while pairs.numel() < want:
        u, v = sample(n * case["deg"] // 2)
        keep = u != v
        u, v = torch.minimum(u, v)[keep], torch.maximum(u, v)[keep]
        pairs = torch.unique(torch.cat([pairs, u * n + v]))
    pairs = pairs[torch.randperm(pairs.numel(), generator=gen, device="cuda")[:want]]
    u, v = pairs // n, pairs % n
    loop = torch.arange(n, device="cuda")
    key = torch.sort(torch.cat([u * n + v, v * n + u, loop * n + loop])).values
    rows = key // n
    row_ptr = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
    row_ptr[1:] = torch.cumsum(torch.bincount(rows, minlength=n), 0)
    return row_ptr, (key - rows * n).to(torch.int32)


def _normal(gen, rows, cols, dtype):
    return torch.randn((rows, cols), generator=gen, device="cuda").to(dtype)


def _glorot(gen, d_in, d_out, dtype):
    lim = math.sqrt(6.0 / (d_in + d_out))
    return ((torch.rand((d_in, d_out), generator=gen, device="cuda") * 2 - 1) * lim).to(dtype)


def _inputs(case, seed):
    """Graph and dense inputs of a case, from the seed alone."""
    gen = _generator(seed)
    kind, n = case["kind"], case["n"]
    dt = DTYPES[case.get("dtype", "f32")]
    s = {}
    if "graph" in case:
        s["csr"] = _csr(case, gen)
    if kind in ("spmm", "attention", "plan"):
        s["X"] = _normal(gen, n, case["d"], dt)
    if kind in ("gcn_layer", "update"):
        s["X"] = _normal(gen, n, case["d_in"], dt)
        s["W"] = _glorot(gen, case["d_in"], case["d_out"], dt)
    if kind in ("step", "gcn_train", "agnn_train"):
        s["X"] = _normal(gen, n, case["d_in"], dt)
        if "gcn" in case:
            s["W1"] = _glorot(gen, case["d_in"], case["gcn"], dt)
            s["W2"] = _glorot(gen, case["gcn"], case["n_out"], dt)
        if "agnn" in case:
            s["Win"] = _glorot(gen, case["d_in"], case["agnn"], dt)
            s["Wout"] = _glorot(gen, case["agnn"], case["n_out"], dt)
    if kind in ("gcn_train", "agnn_train"):
        s["d_out"] = _normal(gen, n, case["n_out"], torch.float32)
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"] = case
    kind, L = case["kind"], B.lib()
    if kind == "update":
        s["out"] = torch.empty((case["n"], case["d_out"]), dtype=torch.float32, device="cuda")
        return s
    g = s["g"] = B.Graph(*s.pop("csr"))
    dt = DTYPES[case.get("dtype", "f32")]
    if kind == "plan":
        s["side"] = B.SideStreams()
        return s
    if kind == "windows":
        s["win"] = B.Windows(g)
        s["win"].win_cols.zero_()  # its capacity is the number of entries, the transformation fills what it needs
        s["ws"] = B._workspace(L.ftc_build_windows_workspace_bytes(g.n, g.nnz, 16, 8), "cuda")
        return s
    if kind == "step":
        s["path"] = HotPath(g, d_feat=case["d_in"], gcn_hidden=case["gcn"], agnn_hidden=case["agnn"], n_out=case["n_out"],
                            agnn_layers=len(BETAS), act_dtype=dt)
        return s
    s["win"] = B.ftc_build_windows(g)
    vals, s["dinv"] = B.ftc_gcn_norm(g, s["win"], want_vals=kind == "spmm")
    if kind == "spmm":
        s["vals"] = vals
        s["out"] = torch.empty((g.n, case["d"]), dtype=torch.float32, device="cuda")
        s["ws"] = B._workspace(L.ftc_spmm_workspace_bytes(g.n, g.nnz, case["d"]), "cuda")
    elif kind == "gcn_layer":
        s["out"] = torch.empty((g.n, case["d_out"]), dtype=torch.float32, device="cuda")
        s["ws"] = B._workspace(L.ftc_gcn_layer_workspace_bytes(g.n, g.nnz, case["d_in"], case["d_out"]), "cuda")
    elif kind == "attention":
        s["out"] = torch.empty((g.n, case["d"]), dtype=torch.float32, device="cuda")
        s["p"] = torch.empty(g.nnz, dtype=torch.float32, device="cuda")
        s["ws"] = B._workspace(L.ftc_agnn_layer_workspace_bytes(g.n, g.nnz, case["d"]), "cuda")
    else:
        s["path"] = TrainPath(g, s["win"], s["dinv"], d_feat=case["d_in"], gcn_hidden=case.get("gcn", 16),
                              agnn_hidden=case.get("agnn", 32), n_out=case["n_out"], agnn_layers=len(BETAS), act_dtype=dt)
    return s


def run(s):
    case, kind = s["case"], s["case"]["kind"]
    if kind == "spmm":
        return B.ftc_spmm(s["g"], s["win"], s["vals"], s["X"], out=s["out"], ws=s["ws"])
    if kind == "update":
        return B.ftc_update_gemm(s["X"], s["W"], out=s["out"])
    if kind == "windows":
        w = B.ftc_build_windows(s["g"], out=s["win"], ws=s["ws"])
        return dict(edge_to_row=w.edge_to_row, edge_to_col=w.edge_to_col, block_partition=w.block_partition,
                    win_col_ptr=w.win_col_ptr, win_cols=w.win_cols, summary=w.summary)
    if kind == "gcn_layer":
        return B.ftc_gcn_layer(s["g"], s["win"], None, s["X"], s["W"], relu=True, out=s["out"], ws=s["ws"], dinv=s["dinv"])
    if kind == "attention":
        out = B.ftc_agnn_layer(s["g"], s["win"], s["X"], beta=case["beta"], out=s["out"], edge_p=s["p"], ws=s["ws"])
        return dict(out=out, p=s["p"])
    if kind == "step":
        path = s["path"]
        path.step(s["X"], s["W1"], s["W2"], s["Win"], s["Wout"], BETAS)
        return dict(gcn=path.gcn_out, agnn=path.agnn_out)
    if kind == "gcn_train":
        path = s["path"]
        out = path.gcn_forward(s["X"], s["W1"], s["W2"])
        dW1, dW2 = path.gcn_backward(s["X"], s["W1"], s["W2"], s["d_out"])
        return dict(out=out, dW1=dW1, dW2=dW2)
    if kind == "agnn_train":
        path = s["path"]
        out = path.agnn_model_forward(s["X"], s["Win"], s["Wout"], BETAS)
        dWin, dWout, dbeta = path.agnn_model_backward(s["X"], s["Win"], s["Wout"], BETAS, s["d_out"])
        return dict(out=out, dWin=dWin, dWout=dWout, dbeta=dbeta)
    plan = PlannedGraph(s["g"], case["d"], DTYPES[case["dtype"]], side=s["side"])
    w = plan.win  # its column lists are as long as the windows want them: "windows" cases return them, in a buffer of fixed size
    return dict(row_ptr=plan.g.row_ptr, col_idx=plan.g.col_idx, edge_to_row=w.edge_to_row, edge_to_col=w.edge_to_col,
                block_partition=w.block_partition, win_col_ptr=w.win_col_ptr, X=plan.enter(s["X"]))


# ---- what a pass cannot do without --------------------------------------------------------------------
def work(case):
    kind, n, e = case["kind"], case["n"], SIZE[case.get("dtype", "f32")]
    if kind == "update":
        d_in, d_out = case["d_in"], case["d_out"]
        return dict(bytes=n * d_in * e + d_in * d_out * e + n * d_out * 4, flops=2 * n * d_in * d_out)
    nnz, rp = _entries(case), 4 * (n + 1)
    graph = 4 * nnz + rp
    index = 8 * nnz + 4 * nnz + 8 * (n // 16)  # rows and positions of the entries, column lists, window arrays
    if kind == "windows":
        return dict(bytes=graph + index, flops=0)
    if kind == "spmm":
        return dict(bytes=graph + 4 * nnz + n * case["d"] * (e + 4), flops=2 * nnz * case["d"])
    if kind == "gcn_layer":
        d_in, d_out = case["d_in"], case["d_out"]
        return dict(bytes=graph + n * (d_in * e + d_out * 4 + 4), flops=2 * n * d_in * d_out + 2 * nnz * d_out)
    if kind == "attention":
        return dict(bytes=graph + 4 * nnz + n * case["d"] * (e + 4), flops=4 * nnz * case["d"])
    if kind == "plan":
        return dict(bytes=2 * graph + index + 2 * n * case["d"] * e, flops=0)
    d_in, n_out, layers = case["d_in"], case["n_out"], len(BETAS)
    gcn = agnn = 0
    if "gcn" in case:
        gcn = 2 * n * d_in * case["gcn"] + 2 * n * case["gcn"] * n_out + 2 * nnz * (case["gcn"] + n_out)
    if "agnn" in case:
        agnn = 2 * n * case["agnn"] * (d_in + n_out) + 4 * layers * nnz * case["agnn"]
    # the graph, the input and the weights once, the outputs once; gradients: the same again
    data = graph + n * d_in * e + (d_in + n_out) * (case.get("gcn", 0) + case.get("agnn", 0)) * e
    if kind == "step":
        return dict(bytes=data + index + 2 * n * n_out * 4, flops=gcn + agnn)
    grads = (d_in + n_out) * (case.get("gcn", 0) + case.get("agnn", 0)) * 4
    return dict(bytes=data + 2 * n * n_out * 4 + grads, flops=(2 * gcn if kind == "gcn_train" else 3 * agnn))


def tolerance(case):
    kind, dtype = case["kind"], case.get("dtype")
    if kind in ("windows", "plan"):
        return "exact"
    if kind == "agnn_train" and dtype != "f32":
        # as below; the gradients of the scalar weights are sums that cancel (seen against 64 bits: 2e-3 in fp16)
        return dict(rel=8e-3 if dtype == "f16" else 6.4e-2)
    if kind in ("step", "gcn_train") and dtype != "f32":
        # activations between the layers are rounded to the type of the inputs (seen against 64 bits: 4e-4 in fp16)
        return dict(rel=2e-3 if dtype == "f16" else 1.6e-2)
    if kind in ("gcn_train", "agnn_train"):
        # a sum near zero that rounds to the other side of the ReLU switches a whole row's share of the weight
        # gradient on or off (seen against 64 bits: 2e-4)
        return dict(rel=1e-3)
    if kind == "gcn_layer" and dtype == "f16":  # the product before the aggregation is kept in fp16 (seen: 2e-4)
        return dict(rel=1e-3)
    return dict(rel=1e-5)  # products of the inputs as they are, summed in 32 bits


# ---- the same in 64 bits --------------------------------------------------------------------------------
class _Exact:
    """Plain fp64 evaluation on one graph; entry-wise work goes in pieces to bound the memory."""

    def __init__(self, csr):
        self.row_ptr, self.cols = csr[0].long(), csr[1].long()
        self.n, self.nnz = self.row_ptr.numel() - 1, self.cols.numel()
        self.deg = self.row_ptr[1:] - self.row_ptr[:-1]
        self.rows = torch.repeat_interleave(torch.arange(self.n, device="cuda"), self.deg)
        self.dinv = self.deg.double().clamp(min=1).rsqrt()

    def pieces(self, d):
        step = max(1, (1 << 26) // max(1, d))
        return [slice(a, min(a + step, self.nnz)) for a in range(0, self.nnz, step)]

    def aggregate(self, vals, X, transposed=False):
        out = torch.zeros((self.n, X.shape[1]), dtype=torch.float64, device="cuda")
        for p in self.pieces(X.shape[1]):
            to, frm = (self.cols[p], self.rows[p]) if transposed else (self.rows[p], self.cols[p])
            out.index_add_(0, to, X[frm] * vals[p, None])
        return out

    def dots(self, X, Y):
        return torch.cat([(X[self.rows[p]] * Y[self.cols[p]]).sum(1) for p in self.pieces(X.shape[1])])

    def row_sum(self, e):
        return torch.zeros(self.n, dtype=torch.float64, device="cuda").index_add_(0, self.rows, e)

    def gcn_vals(self):
        return self.dinv[self.rows] * self.dinv[self.cols]

    def attention(self, H, beta):
        norm = H.norm(dim=1).clamp(min=1e-12)
        cos = self.dots(H / norm[:, None], H / norm[:, None])
        p = torch.exp(beta * cos - abs(beta))
        p = p / self.row_sum(p)[self.rows]
        return self.aggregate(p, H), p, cos, norm

    def attention_backward(self, H, beta, p, cos, norm, dY):
        hn = H / norm[:, None]
        dp = self.dots(dY, H)
        ds = p * (dp - self.row_sum(p * dp)[self.rows])
        q = beta * (self.aggregate(ds, hn) + self.aggregate(ds, hn, transposed=True))
        dH = self.aggregate(p, dY, transposed=True) + (q - hn * (hn * q).sum(1, keepdim=True)) / norm[:, None]
        return dH, (ds * cos).sum()


def _exact_windows(csr, n):
    """The graph transformation with 16-row windows and 8-column blocks, as sorted distinct (window, column) pairs."""
    row_ptr, cols = csr[0].long(), csr[1].long()
    rows = torch.repeat_interleave(torch.arange(n, device="cuda"), row_ptr[1:] - row_ptr[:-1])
    n_win = (n + 15) // 16
    pairs, where = torch.unique((rows // 16) * n + cols, return_inverse=True)
    counts = torch.bincount(pairs // n, minlength=n_win)
    start = torch.zeros(n_win + 1, dtype=torch.int64, device="cuda")
    start[1:] = torch.cumsum(counts, 0)
    blocks = (counts + 7) // 8
    i32 = lambda t: t.to(torch.int32)
    return dict(edge_to_row=i32(rows), edge_to_col=i32(where - start[rows // 16]), block_partition=i32(blocks),
                win_col_ptr=i32(start), win_cols=i32(pairs % n)), torch.stack([counts.sum(), blocks.sum()])


def _exact_relabel(csr, n, perm):
    row_ptr, cols = csr[0].long(), csr[1].long()
    deg = row_ptr[1:] - row_ptr[:-1]
    rows = torch.repeat_interleave(torch.arange(n, device="cuda"), deg)
    inv = torch.empty_like(perm)
    inv[perm] = torch.arange(n, device="cuda")
    key = torch.sort(inv[rows] * n + inv[cols]).values
    new_ptr = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
    new_ptr[1:] = torch.cumsum(deg[perm], 0)
    return new_ptr, (key % n).to(torch.int32)


def _exact_labels(csr, n, rounds):
    """Synchronous label propagation: the most frequent label of the row's entries, the smallest on a tie."""
    row_ptr, cols = csr[0].long(), csr[1].long()
    rows = torch.repeat_interleave(torch.arange(n, device="cuda"), row_ptr[1:] - row_ptr[:-1])
    labels = torch.arange(n, device="cuda")
    for _ in range(rounds):
        pairs, votes = torch.unique(rows * n + labels[cols], return_counts=True)
        best = torch.zeros(n, dtype=torch.int64, device="cuda")
        best.scatter_reduce_(0, pairs // n, votes * n + (n - 1 - pairs % n), "amax")
        labels = n - 1 - best % n
    return labels


def _exact_plan(case, s):
    n, csr = case["n"], s["csr"]
    win, summary = _exact_windows(csr, n)
    X, deg, nnz = s["X"], (csr[0][1:] - csr[0][:-1]).long(), csr[1].numel()
    perm = None
    if n * case["d"] * SIZE[case["dtype"]] > 4 * 1024 * 1024:  # a feature matrix larger than one L2
        if n * float((deg * deg).sum()) / nnz ** 2 >= 2.0:
            classes = torch.floor(torch.log2(deg.double())) + 1
            perm = torch.sort(-classes, stable=True).indices
        elif nnz >= 8 * n:
            perm = torch.sort(_exact_labels(csr, n, 10), stable=True).indices
            trial = _exact_windows(_exact_relabel(csr, n, perm), n)[1]
            if int(trial[0]) > 0.98 * int(summary[0]):
                perm = None
    if perm is not None:
        csr = _exact_relabel(csr, n, perm)
        win, X = _exact_windows(csr, n)[0], X[perm]
    del win["win_cols"]
    return dict(row_ptr=csr[0], col_idx=csr[1], X=X, **win)


def exact(case, seed):
    s = _inputs(case, seed)
    kind = case["kind"]
    if kind == "plan":
        return _exact_plan(case, s)
    if kind == "windows":
        win, summary = _exact_windows(s["csr"], case["n"])
        cols = torch.zeros(s["csr"][1].numel(), dtype=torch.int32, device="cuda")
        cols[:win["win_cols"].numel()] = win["win_cols"]
        return dict(win, win_cols=cols, summary=summary)
    f = {k: t.double() for k, t in s.items() if k != "csr"}
    if kind == "update":
        return f["X"] @ f["W"]
    G = _Exact(s["csr"])
    if kind == "spmm":
        return G.aggregate(G.gcn_vals(), f["X"])
    if kind == "gcn_layer":
        return torch.relu(G.aggregate(G.gcn_vals(), f["X"] @ f["W"]))
    if kind == "attention":
        out, p = G.attention(f["X"], case["beta"])[:2]
        return dict(out=out, p=p)
    r = {}
    if kind in ("step", "gcn_train"):
        A = G.gcn_vals()
        h = torch.relu(G.aggregate(A, f["X"] @ f["W1"]))
        out = G.aggregate(A, h @ f["W2"])
        if kind == "step":
            r["gcn"] = out
        else:  # the operator is symmetric
            dZ2 = G.aggregate(A, f["d_out"])
            dZ1 = G.aggregate(A, (dZ2 @ f["W2"].T) * (h > 0))
            return dict(out=out, dW1=f["X"].T @ dZ1, dW2=h.T @ dZ2)
    H, kept = torch.relu(f["X"] @ f["Win"]), []
    for beta in BETAS:
        Y, p, cos, norm = G.attention(H, beta)
        kept.append((H, p, cos, norm))
        H = Y
    out = H @ f["Wout"]
    if kind == "step":
        return dict(r, agnn=out)
    dWout, d, dbeta = H.T @ f["d_out"], f["d_out"] @ f["Wout"].T, [None] * len(BETAS)
    for l in reversed(range(len(BETAS))):
        Hl, p, cos, norm = kept[l]
        d, dbeta[l] = G.attention_backward(Hl, BETAS[l], p, cos, norm, d)
    return dict(out=out, dWin=f["X"].T @ (d * (kept[0][0] > 0)), dWout=dWout, dbeta=torch.stack(dbeta))
