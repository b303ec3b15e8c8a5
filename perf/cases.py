"""The workloads this library is timed on: what they are, their inputs, one pass through the public entry points, and the
work and the rounding error a pass has.

A case is one GNN workload: a synthetic graph, one or two layers and a direction (inference, or a training iteration = forward and
backward).  Graphs, layer widths and distributions are those of the benchmark and of the tests (Erdos-Renyi, R-MAT and thinned-grid
patterns with self loops, sampled mini-batch blocks; X uniform in [-1, 1], Glorot-uniform weights, attention vectors normal(0, 0.1)).
All arithmetic is fp32, the one data type of the library.
"""
from __future__ import annotations

import math

import torch

from paper_2306_15155_amd import ACT_NONE, ACT_RELU, KIND_GAT, KIND_GCN, SELECT_MODEL, Context, Panels, Tiles, csr_struct

DEV = "cuda:0"
SLOPE = 0.2


def _case(name, task, graph, nodes, pairs, f_in, f_hid, f_out, heads=1, hops=0):
    c = {"task": task, "graph": graph, "nodes": nodes, "pairs": pairs, "f_in": f_in, "f_hid": f_hid, "f_out": f_out, "heads": heads, "hops": hops}
    return dict(c, name=name) if name else c


def listed():
    """graph: er / rmat = that many distinct undirected `pairs` between `nodes` nodes, mirrored, plus self loops; grid = a square grid of
    about `nodes` nodes with `pairs` of its links kept; blocks = `nodes` seed nodes sampled from an R-MAT graph of 2.45 M nodes and
    `pairs` pairs.  f_hid = 0: one layer f_in -> f_out, otherwise f_in -> f_hid (ReLU) -> f_out."""
    return [
        # the smallest call: one GCN layer on a 10,000-node graph, where launches and host time are all there is
        _case("er10k_gcn_infer", "gcn_infer", "er", 10_000, 50_000, 64, 0, 32),
        # serving with neighbour sampling: two GCN layers over the blocks of 1,024 seeds with fan-outs 10 and 25
        _case("blocks_gcn_infer", "gcn_infer", "blocks", 1024, 62_250_000, 100, 256, 47),
        # the same blocks in mini-batch training
        _case("blocks_gcn_train", "gcn_train", "blocks", 1024, 62_250_000, 100, 256, 47),
        # ordinary sizes: a citation- or product-graph-sized pattern (100,000 nodes, about 20 entries per row) in training, one case per
        # layer family beside plain GCN: multi-head attention, GATv2, the K-hop layers
        _case("rmat100k_gat4_train", "gat_train", "rmat", 100_000, 1_000_000, 128, 0, 128, heads=4),
        _case("rmat50k_gatv2_train", "gatv2_train", "rmat", 50_000, 1_500_000, 100, 0, 64),
        _case("rmat100k_tagcn_train", "tagcn_train", "rmat", 100_000, 1_000_000, 100, 0, 47, hops=2),
        # the benchmark's own step on the dense power-law graph of a social network (115 M entries, hubs): two GCN layers and a GAT layer
        _case("rmat233k_step", "step", "rmat", 233_000, 57_471_634, 602, 256, 41),
        # training on that graph: the paper's evaluation trains both models
        _case("rmat233k_gcn_train", "gcn_train", "rmat", 233_000, 57_471_634, 602, 256, 41),
        _case("rmat233k_gat_train", "gat_train", "rmat", 233_000, 57_471_634, 602, 0, 256),
        # ten times the nodes at a tenth of the degree (a co-purchase graph), hidden size 512: the largest case
        _case("rmat2450k_gcn_infer", "gcn_infer", "rmat", 2_450_000, 62_250_000, 100, 512, 512),
        # a road network: 12 M nodes, three entries per row, no hubs
        _case("grid12m_gcn_infer", "gcn_infer", "grid", 11_999_296, 12_700_000, 128, 32, 128),
        # the densest graph of the paper's table: 98,000 nodes, 1,021 entries per row, no hubs
        _case("er98k_gat_infer", "gat_infer", "er", 98_000, 50_000_000, 64, 0, 256),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    task = rng.choice(("gcn_infer", "gcn_infer", "gcn_train", "gcn_train", "gat_infer", "gat_train", "gat_train", "sgc_train", "tagcn_train",
                       "gatv2_train", "dotgat_train"))
    two = task in ("gcn_infer", "gcn_train") and rng.random() < 0.7
    graph = rng.choice(("er", "rmat", "rmat", "grid", "blocks") if two else ("er", "rmat", "rmat", "grid"))
    heads, hops = 1, 0
    f_in, f_hid = _logint(rng, 16, 608), _logint(rng, 16, 320) if two else 0
    f_out = _logint(rng, 8, 256)
    if task in ("gat_infer", "gat_train") and rng.random() < 0.5:
        heads = rng.choice((2, 4, 8))
        f_out = heads * _logint(rng, 8, 64)
    if task in ("sgc_train", "tagcn_train"):
        hops = rng.choice((2, 3))
    if graph == "blocks":
        return _case(None, task, graph, _logint(rng, 128, 4096), 62_250_000, f_in, f_hid, f_out)
    n = _logint(rng, 2_000, 2_400_000)
    if graph == "grid":
        side = int(math.sqrt(n))
        return _case(None, task, graph, side * side, int(2 * side * (side - 1) * rng.uniform(0.5, 0.95)), f_in, f_hid, f_out, heads, hops)
    # entries times width bounded so that no drawn case costs more than the largest listed one
    width = max(f_in, f_hid, f_out)
    budget = {"gcn_infer": 3e10, "gcn_train": 1.2e10, "gat_infer": 1.2e10, "gat_train": 5e9}.get(task, 2.5e9)
    degree = min(_logint(rng, 4, 600), n // 20, int(1e8) // n, max(4, int(budget / (width * n))))
    return _case(None, task, graph, n, n * max(degree, 2) // 2, f_in, f_hid, f_out, heads, hops)


# ------------------------------------------------------------------------------------------------------------------------- inputs

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(1_000_003 * (int(seed) + 1))
    return g


def _csr(keys, n_rows, n_cols):
    """Canonical CSR (int32) of sorted distinct keys row * n_cols + col."""
    rows = torch.div(keys, n_cols, rounding_mode="floor")
    cols = (keys - rows * n_cols).to(torch.int32)
    ptr = torch.zeros(n_rows + 1, dtype=torch.int64, device=DEV)
    ptr[1:] = torch.cumsum(torch.bincount(rows, minlength=n_rows), 0)
    return ptr.to(torch.int32), cols


def _mirrored(pair_keys, n):
    u = torch.div(pair_keys, n, rounding_mode="floor")
    v = pair_keys - u * n
    i = torch.arange(n, device=DEV)
    return _csr(torch.sort(torch.cat([pair_keys, v * n + u, i * (n + 1)]))[0], n, n)


def _rmat_pairs(g, n, m):
    """m draws of R-MAT(0.57, 0.19, 0.19, 0.05) on ceil(log2 n) levels as keys min * n + max; loops and draws out of range dropped."""
    u = torch.zeros(m, dtype=torch.int64, device=DEV)
    v = torch.zeros(m, dtype=torch.int64, device=DEV)
    for _ in range(max(1, math.ceil(math.log2(n)))):
        x = torch.rand(m, generator=g, device=DEV)
        u.mul_(2).add_(x >= 0.76)
        v.mul_(2).add_(((x >= 0.57) & (x < 0.76)) | (x >= 0.95))
    ok = (u < n) & (v < n) & (u != v)
    u, v = u[ok], v[ok]
    return torch.minimum(u, v) * n + torch.maximum(u, v)


def _er_pairs(g, n, m):
    u = torch.randint(0, n, (m,), generator=g, device=DEV)
    v = torch.randint(0, n, (m,), generator=g, device=DEV)
    u, v = u[u != v], v[u != v]
    return torch.minimum(u, v) * n + torch.maximum(u, v)


def _graph(g, kind, n, pairs):
    """The pattern with exactly `pairs` distinct undirected links (a uniform choice among those drawn), mirrored, with self loops."""
    if kind == "grid":
        side = math.isqrt(n)
        i = torch.arange(n, device=DEV)
        right, down = i[i % side != side - 1], i[: n - side]
        keys = torch.cat([right * n + right + 1, down * n + down + side])
    else:
        keys = torch.empty(0, dtype=torch.int64, device=DEV)
        m, tries = int(pairs * (1.35 if kind == "rmat" else 1.02)) + 64, 0
        while keys.numel() < pairs and tries < 40:
            keys = torch.unique(torch.cat([keys, (_rmat_pairs if kind == "rmat" else _er_pairs)(g, n, m)]))
            m, tries = max(2 * (pairs - keys.numel()), pairs // 16) + 64, tries + 1
        if keys.numel() < pairs:
            raise ValueError(f"{pairs} distinct links not reached on {n} nodes")
    keys = keys[torch.randperm(keys.numel(), generator=g, device=DEV)[:pairs]]
    return _mirrored(keys, n)


def _sample(g, row_ptr, col_idx, dst, fanout, n):
    """One hop of fan-out sampling without replacement -> (rows, cols) of the block in local numbering with self edges, global column ids;
    the destinations are the first columns."""
    lo, deg = row_ptr[dst].long(), (row_ptr[dst + 1] - row_ptr[dst]).long()
    row = torch.repeat_interleave(torch.arange(dst.numel(), device=DEV), deg)
    col = col_idx[torch.arange(row.numel(), device=DEV) - torch.repeat_interleave(torch.cumsum(deg, 0) - deg - lo, deg)].long()
    row, col = row[col != dst[row]], col[col != dst[row]]
    order = torch.argsort(row.double() + torch.rand(row.numel(), generator=g, device=DEV, dtype=torch.float64))
    row, col = row[order], col[order]
    count = torch.bincount(row, minlength=dst.numel())
    keep = torch.arange(row.numel(), device=DEV) - (torch.cumsum(count, 0) - count)[row] < fanout
    row, col = row[keep], col[keep]
    local = torch.full((n,), -1, dtype=torch.int64, device=DEV)
    local[dst] = torch.arange(dst.numel(), device=DEV)
    fresh = torch.unique(col[local[col] < 0])
    local[fresh] = torch.arange(fresh.numel(), device=DEV) + dst.numel()
    self_edge = torch.arange(dst.numel(), device=DEV)
    return torch.cat([row, self_edge]), torch.cat([local[col], self_edge]), torch.cat([dst, fresh])


class _Pattern:
    """A pattern, its transpose (itself when symmetric), the normalisation vectors and the layout the library advises for it."""

    def __init__(self, ctx, n_rows, n_cols, row_ptr, col_idx, transposed=None, widest=0):
        self.n_rows, self.n_cols, self.nnz = n_rows, n_cols, col_idx.numel()
        args = (n_rows, n_cols, row_ptr, col_idx)
        A = csr_struct(*args)
        deg_r, deg_c = ctx.degrees(A)
        self.r, self.c = ctx.norm_vectors(deg_r), ctx.norm_vectors(deg_c)
        layout = {}
        if widest and self.nnz >= 1_000_000:     # once per graph: the dense-tile split where it pays, else measured column panels
            tiles = Tiles(ctx, A, 0.07, (widest + 31) // 32 * 32)
            if tiles.nnz_dense * 3 >= self.nnz:
                layout = {"tiles": tiles}
            else:
                tiles.close()
                del tiles
                panels = Panels(ctx, A, 0, tune=True)
                layout = {"panels": panels} if panels.count > 1 else {}
        self.A = csr_struct(*args, **layout)
        self.At = self.A if transposed is None else csr_struct(n_cols, n_rows, *transposed)
        self.val = None
        self._args, self._layout = args, layout

    def for_composition(self, ctx, comp):
        """PRE_* compositions take the pattern with the values of the normalised adjacency."""
        if comp < 4:
            return self.A
        if self.val is None:
            self.val = ctx.gcn_precompute(self.A, self.r, self.c)
            self.Apre = csr_struct(*self._args, self.val, **self._layout)
        return self.Apre


def _uniform(g, *shape, bound=1.0):
    return torch.empty(shape, device=DEV).uniform_(-bound, bound, generator=g)


def _glorot(g, f_in, f_out, blocks=1):
    return _uniform(g, blocks * f_in, f_out, bound=math.sqrt(6.0 / (f_in + f_out)))


def _normal(g, *shape, std=1.0):
    return torch.empty(shape, device=DEV).normal_(0.0, std, generator=g)


def _layers(case):
    return [(case["f_in"], case["f_hid"]), (case["f_hid"], case["f_out"])] if case["f_hid"] else [(case["f_in"], case["f_out"])]


def prepare(case, seed):
    g, ctx = _gen(seed), Context(0)
    task, layers = case["task"], _layers(case)
    gcn_like = task in ("gcn_infer", "gcn_train", "step", "sgc_train", "tagcn_train")
    if case["graph"] == "blocks":
        n = 2_450_000
        row_ptr, col_idx = _graph(g, "rmat", n, case["pairs"])
        ids = torch.randperm(n, generator=g, device=DEV)[: case["nodes"]]
        patterns = []
        for fanout in (10, 25):
            rows, cols, src = _sample(g, row_ptr, col_idx, ids, fanout, n)
            nr, nc = ids.numel(), src.numel()
            csr = _csr(torch.sort(rows * nc + cols)[0], nr, nc)
            csr_t = _csr(torch.sort(cols * nr + rows)[0], nc, nr)
            patterns.insert(0, _Pattern(ctx, nr, nc, *csr, transposed=csr_t))
            ids = src
        n_src = ids.numel()
        del row_ptr, col_idx
    else:
        row_ptr, col_idx = _graph(g, case["graph"], case["nodes"], case["pairs"])
        n_src = case["nodes"]
        widest = max(min(w) for w in layers) if gcn_like else case["f_out"] if task in ("gat_infer", "gat_train") else 0
        if task == "step":
            widest = max(case["f_hid"], widest)
        patterns = [_Pattern(ctx, n_src, n_src, row_ptr, col_idx, widest=widest)] * len(layers)
    s = {"ctx": ctx, "task": task, "heads": case["heads"], "hops": case["hops"], "patterns": patterns, "X": _uniform(g, n_src, case["f_in"])}
    p0, last = patterns[0], patterns[-1]
    f_in, f_out = layers[0][0], layers[-1][1]
    train = task.endswith("_train")
    if train:
        s["dY"] = _normal(g, last.n_rows, f_out)
    if task in ("gcn_infer", "gcn_train", "step"):
        s["W"] = [_glorot(g, *w) for w in layers]
        s["comp"] = [ctx.select(KIND_GCN, p.A, *w, SELECT_MODEL)[0] for p, w in zip(patterns, layers)]
        s["csr"] = [p.for_composition(ctx, k) for p, k in zip(patterns, s["comp"])]
        if train:
            s["bwd"] = [ctx.select_gcn_backward(p.A, *w, want_dx=i > 0)[0] for i, (p, w) in enumerate(zip(patterns, layers))]
    if task in ("gat_infer", "gat_train", "step"):
        width = case["f_hid"] if task == "step" else f_out
        s["Wg"], s["a_l"], s["a_r"] = _glorot(g, f_in, width), _normal(g, width, std=0.1), _normal(g, width, std=0.1)
        s["gat_comp"] = ctx.select(KIND_GAT, p0.A, f_in, width, SELECT_MODEL)[0]
    if task in ("sgc_train", "tagcn_train"):
        s["W"] = _glorot(g, f_in, f_out, case["hops"] + 1 if task == "tagcn_train" else 1)
        s["comp"] = 0 if f_in <= f_out else 1
        s["bwd"] = ctx.select_khop_backward(p0.A, f_in, f_out, case["hops"], task == "tagcn_train")[0]
    if task == "gatv2_train":
        s["W"], s["att"], s["comp"] = [_glorot(g, f_in, f_out) for _ in range(2)], _normal(g, f_out, std=0.1), 1 if f_in < f_out else 0
    if task == "dotgat_train":
        d_k = min(64, f_out)
        s["W"] = [_glorot(g, f_in, d_k), _glorot(g, f_in, d_k), _glorot(g, f_in, f_out)]
        s["scale"], s["comp"] = 1.0 / math.sqrt(d_k), 1 if f_in < f_out else 0
    if task in ("gat_train", "gatv2_train", "dotgat_train"):
        s["t_pos"] = ctx.transpose_positions(p0.A, p0.At)
    return s


# ------------------------------------------------------------------------------------------------------------------------ one pass

def _gcn_forward(s):
    outs, x = [], s["X"]
    for i, p in enumerate(s["patterns"]):
        act = ACT_RELU if i + 1 < len(s["patterns"]) or s["task"] == "gcn_infer" and i == 0 else ACT_NONE
        x = s["ctx"].gcn_layer(s["csr"][i], p.r, p.c, x, s["W"][i], s["comp"][i], act)
        outs.append(x)
    return outs


def _gcn_backward(s, outs):
    grads, dY, last = [], s["dY"], len(outs) - 1
    for i in range(last, -1, -1):
        p, relu = s["patterns"][i], i < last
        dY, dW = s["ctx"].gcn_backward(p.A, p.At, p.r, p.c, outs[i - 1] if i else s["X"], s["W"][i], dY, s["bwd"][i],
                                       Y=outs[i] if relu else None, activation=ACT_RELU if relu else ACT_NONE, want_dx=i > 0)
        grads.append(dW)
    return grads


def _gat_forward(s):
    A = s["patterns"][0].A
    if s["heads"] == 1:
        return s["ctx"].gat_layer(A, s["X"], s["Wg"], s["a_l"], s["a_r"], s["gat_comp"], SLOPE, ACT_RELU)
    return s["ctx"].gat_layer_heads(A, s["X"], s["Wg"], s["a_l"], s["a_r"], s["heads"], s["gat_comp"], SLOPE, ACT_RELU)


def run(s):
    ctx, task, p, X = s["ctx"], s["task"], s["patterns"][0], s["X"]
    if task == "gcn_infer":
        return _gcn_forward(s)[-1]
    if task == "gcn_train":
        outs = _gcn_forward(s)
        return outs[-1], _gcn_backward(s, outs)
    if task == "step":
        return _gcn_forward(s)[-1], _gat_forward(s)
    if task == "gat_infer":
        return _gat_forward(s)
    if task == "gat_train":
        Y = _gat_forward(s)
        if s["heads"] == 1:
            return Y, ctx.gat_backward(p.A, p.At, s["t_pos"], X, s["Wg"], s["a_l"], s["a_r"], s["dY"], Y=Y, neg_slope=SLOPE, activation=ACT_RELU)
        return Y, ctx.gat_backward_heads(p.A, p.At, s["t_pos"], X, s["Wg"], s["a_l"], s["a_r"], s["heads"], s["dY"], Y=Y, neg_slope=SLOPE,
                                         activation=ACT_RELU)
    # the other layers train as a model's only layer: linear outputs
    if task == "sgc_train":
        Y = ctx.sgc_layer(p.A, p.r, p.c, X, s["W"], s["hops"], s["comp"])
        return Y, ctx.sgc_backward(p.A, p.At, p.r, p.c, X, s["W"], s["hops"], s["dY"], s["bwd"])
    if task == "tagcn_train":
        Y = ctx.tagcn_layer(p.A, p.r, p.c, X, s["W"], s["hops"], s["comp"])
        return Y, ctx.tagcn_backward(p.A, p.At, p.r, p.c, X, s["W"], s["hops"], s["dY"], s["bwd"])
    if task == "gatv2_train":
        Y = ctx.gatv2_layer(p.A, X, s["W"][0], s["W"][1], s["att"], s["comp"], SLOPE)
        return Y, ctx.gatv2_backward(p.A, p.At, s["t_pos"], X, s["W"][0], s["W"][1], s["att"], s["dY"], neg_slope=SLOPE)
    if task == "dotgat_train":
        Y = ctx.dotgat_layer(p.A, X, *s["W"], s["scale"], s["comp"])
        return Y, ctx.dotgat_backward(p.A, p.At, s["t_pos"], X, *s["W"], s["scale"], s["dY"])
    raise ValueError(task)


# ------------------------------------------------------------------------------------------------------------- work and tolerance

def work(case):
    """Bytes: every operand of every layer call read once, every result written once.  Operations: the products with the weights and
    the sums over the stored entries at the narrower width of the layer."""
    task, layers = case["task"], _layers(case)
    train = task.endswith("_train")
    if case["graph"] == "blocks":    # rows and entries per seed of the sampled blocks (means; a third of the rows has under three neighbours)
        n = case["nodes"]
        shapes = [(4.75 * n, 62 * n, 103 * n), (n, 4.75 * n, 5.1 * n)]
    else:
        shapes = [(case["nodes"], case["nodes"], 2 * case["pairs"] + case["nodes"])] * len(layers)
    calls = [(shape, w, max(case["hops"], 1)) for shape, w in zip(shapes, layers)]
    if task == "step":
        calls.append((shapes[0], layers[0], 1))
    total_bytes = total_flops = 0.0
    for i, ((nr, nc, nnz), (fi, fo), hops) in enumerate(calls):
        blocks = hops + 1 if task == "tagcn_train" else 2 if task == "gatv2_train" else 3 if task == "dotgat_train" else 1
        pattern, x, y, w = 4.0 * (nnz + nr + nc), 4.0 * nc * fi, 4.0 * nr * fo, 4.0 * blocks * fi * fo
        gemm, agg = 2.0 * blocks * min(nr, nc) * fi * fo, 2.0 * hops * nnz * min(fi, fo)
        total_bytes += pattern + x + w + y
        total_flops += gemm + agg
        if train:
            dx = case["f_hid"] == 0 or i > 0
            total_bytes += pattern + x + w + 2 * y + w + (x if dx else 0)
            total_flops += gemm * (2 if dx else 1) + agg * (2 if task in ("gat_train", "gatv2_train", "dotgat_train") else 1)
    return {"bytes": total_bytes, "flops": total_flops}


def tolerance(case):
    """Four times the largest difference between a pass and the same pass with its sums in another order (other composition, no split or
    panels, nodes and features renumbered).  Linear layers and forward passes are smooth: fp32 rounding only.  Where a derivative jumps at
    zero (ReLU of a hidden layer, the LeakyReLU of a GATv2 score) a few values per million lie within rounding of the jump and take the
    other branch, which moves the gradient rows they belong to: far outliers (max) and a 2-norm in the 1e-4 to 1e-3 range."""
    if case["task"] == "gat_train":
        return {"rel": 5e-3, "max": 0.95}     # measured 1.3e-3, 0.36
    if case["task"] == "gatv2_train":
        return {"rel": 6e-3, "max": 0.35}     # measured 1.6e-3, 8.3e-2
    if case["task"] == "gcn_train" and case["f_hid"]:
        return {"rel": 4.5e-3, "max": 0.12}   # measured 1.1e-3, 3.0e-2
    return {"rel": 3.5e-6, "max": 6e-5}       # measured 8.7e-7, 1.5e-5
