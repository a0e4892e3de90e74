"""Performance cases: the work a user of this framework has it do, through its public entry points.

Kinds (field "kind" of a case) and what each stands for:
  step    one training step of a MaskedGNN on a partition that is already on the GPU (active sets, forward pass, loss,
          backward pass): what a training loop repeats
  agg     one masked neighbour aggregation of a layer, forward (its input gathered for the rows of the layer) or
          backward (the output gradient gathered over the transposed graph, cut to the forward rows)
  linear  the feature transform of a layer: forward with bias and ReLU, or backward (weight and bias gradients, then
          the input gradient masked by the ReLU below)
  norm    pre-activation of a layer of the deep residual model, forward and backward
  extract what a program does once per partition: active sets of the unpartitioned graph, extraction of the local graph
  sample  expansion-aware sampling of a partition's boundary, and extraction of the sampled partition
  mask    a layer's edge mask of layer-wise sampling, and the same mask for the backward pass; rebuilt in every step

Graphs are symmetric, column-sorted and seeded: Chung-Lu with exponent 2.1 (every workload of the benchmark but the
toy) or Erdos-Renyi, made on the GPU; partitions are grown breadth-first from a random vertex, extracted and numbered
by the framework itself, as its benchmark does.
"""
import math

import torch

import paper_2311_06837_amd as P

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}


# ---- the cases -------------------------------------------------------------------------------------------------
def listed():
    return [
        # the toy workload, the smallest thing anybody trains: launches and latency
        {"name": "step_toy_gcn_f32", "kind": "step", "graph": "er", "n": 10_000, "deg": 10, "model": "gcn", "dtype": "f32",
         "dims": "64-64-8", "frac": 0.2},
        # the headline workload: 3-layer GraphSAGE of Reddit's shape
        {"name": "step_reddit_sage_f32", "kind": "step", "graph": "cl", "n": 233_000, "deg": 490, "model": "sage", "dtype": "f32",
         "dims": "602-256-256-41", "frac": 0.125},
        # an inner layer of the 8-layer bf16 model: short rows, mean
        {"name": "agg_fwd_bf16_128", "kind": "agg", "dir": "fwd", "n": 1_000_000, "deg": 20, "F": 128, "dtype": "bf16", "model": "sage",
         "frac": 0.0625, "hops": 2},
        # the backward aggregation of a hidden layer, rows cut to the layer's own
        {"name": "agg_bwd_bf16_256", "kind": "agg", "dir": "bwd", "n": 2_000_000, "deg": 15, "F": 256, "dtype": "bf16", "model": "sage",
         "frac": 0.125, "hops": 2},
        # the hidden layer of the products-like GCN: 1 KB rows, symmetric normalisation
        {"name": "agg_fwd_f32_256", "kind": "agg", "dir": "fwd", "n": 1_200_000, "deg": 50, "F": 256, "dtype": "f32", "model": "gcn",
         "frac": 0.125, "hops": 2},
        # its input layer: 100 features, the whole graph
        {"name": "agg_fwd_f32_100", "kind": "agg", "dir": "fwd", "n": 2_450_000, "deg": 50, "F": 100, "dtype": "f32", "model": "gcn",
         "frac": 0.125, "hops": 3},
        # feature transform of a hidden GraphSAGE layer
        {"name": "linear_fwd_f32_256", "kind": "linear", "dir": "fwd", "M": 600_001, "K": 256, "N": 256, "src": 2, "dtype": "f32", "up": 1.0},
        # its backward pass in bf16 (sampled-partition workload)
        {"name": "linear_bwd_bf16_256", "kind": "linear", "dir": "bwd", "M": 900_007, "K": 256, "N": 256, "src": 2, "dtype": "bf16", "up": 1.3},
        # pre-activation of the residual model at its middle width
        {"name": "norm_bf16_256", "kind": "norm", "M": 1_000_000, "F": 256, "dtype": "bf16", "up": 1.0},
        # partition of the 8-layer workload, eight rings
        {"name": "extract_8_hops", "kind": "extract", "n": 1_000_000, "deg": 20, "frac": 0.0625, "hops": 8},
        # boundary sampling at the paper's setting, fanout 5
        {"name": "sample_fanout_5", "kind": "sample", "n": 5_000_000, "deg": 15, "frac": 0.125, "fanout": 5},
        # layer-wise sampling, 10 neighbours a row
        {"name": "mask_fanout_10", "kind": "mask", "n": 1_200_000, "deg": 50, "rule": "fanout", "fanout": 10, "frac": 0.125, "hops": 2},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _graph_size(rng, n_lo, n_hi, deg_lo, deg_hi, most):
    n = _log(rng, n_lo, n_hi)
    deg = _log(rng, deg_lo, min(deg_hi, max(deg_lo, n // 20)))
    return max(n_lo, min(n, most // deg)), deg


def draw(rng):
    kind = rng.choice(["step", "agg", "agg", "agg", "linear", "linear", "norm", "extract", "sample", "mask"])
    dtype = rng.choice(["f32", "bf16"])
    model = rng.choice(["gcn", "sage"])
    frac = round(rng.uniform(0.05, 0.3), 3)
    if kind == "step":       # fp32 only: with 16-bit storage a change of rounding travels through every layer behind it
        n, deg = _graph_size(rng, 5_000, 400_000, 5, 300, 30_000_000)
        hidden = rng.choice([64, 128, 200, 256])
        dims = [rng.choice([64, 100, 128, 602])] + [hidden] * rng.choice([1, 2]) + [rng.choice([8, 16, 41, 47])]
        return {"kind": kind, "graph": rng.choice(["er", "cl", "cl"]), "n": n, "deg": deg, "model": model, "dtype": "f32",
                "dims": "-".join(str(d) for d in dims), "frac": frac}
    if kind == "agg":
        n, deg = _graph_size(rng, 10_000, 2_500_000, 5, 400, 60_000_000)
        F = rng.choice([16, 41, 47, 64, 100, 128, 128, 256, 256, 512, 602, rng.randint(8, 640)])
        return {"kind": kind, "dir": rng.choice(["fwd", "bwd"]), "n": n, "deg": deg, "F": F, "dtype": dtype, "model": model, "frac": frac,
                "hops": rng.choice([1, 2, 3])}
    if kind == "linear":
        M = _log(rng, 2_000, 1_200_000)
        K = rng.choice([64, 100, 128, 256, 256, 512, 602, rng.randint(33, 640)])
        N = rng.choice([16, 41, 47, 64, 128, 256, 256, 512, rng.randint(8, 300)])
        return {"kind": kind, "dir": rng.choice(["fwd", "bwd"]), "M": M, "K": K, "N": N, "src": 2 if model == "sage" else 1, "dtype": dtype,
                "up": round(rng.uniform(1.0, 2.0), 2)}
    if kind == "norm":
        F = rng.choice([64, 128, 256, 512, rng.randint(20, 1000)])
        return {"kind": kind, "M": min(_log(rng, 5_000, 2_000_000), 400_000_000 // F), "F": F, "dtype": dtype, "up": round(rng.uniform(1.0, 1.5), 2)}
    if kind == "extract":
        n, deg = _graph_size(rng, 20_000, 3_000_000, 5, 200, 60_000_000)
        return {"kind": kind, "n": n, "deg": deg, "frac": frac, "hops": rng.choice([1, 2, 3, 5, 8])}
    if kind == "sample":
        n, deg = _graph_size(rng, 50_000, 6_000_000, 5, 100, 70_000_000)
        return {"kind": kind, "n": n, "deg": deg, "frac": frac, "fanout": rng.choice([1, 3, 5, 10, 15, 25])}
    n, deg = _graph_size(rng, 20_000, 2_000_000, 5, 200, 60_000_000)
    return {"kind": kind, "n": n, "deg": deg, "rule": rng.choice(["fanout", "fanout", "threshold"]), "fanout": rng.choice([2, 5, 10, 15, 25]),
            "frac": frac, "hops": rng.choice([1, 2, 3])}


# ---- seeded inputs, made on the GPU ---------------------------------------------------------------------------
# A case's graph and partition have one structure, drawn from its sizes; a seed names the vertices (a permutation of the
# ids) and makes the values.  So the sizes of all outputs belong to the case.
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _csr(keys, n):
    """Sorted distinct keys row * n + column -> Graph."""
    row = keys // n
    row_ptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    row_ptr[1:] = torch.cumsum(torch.bincount(row, minlength=n), 0)
    return P.Graph(row_ptr.int(), (keys - row * n).int(), sorted_columns=True)


def _structure(case, self_loops):
    """Keys of a symmetric random graph without repeated entries, about n * deg of them."""
    n, want = case["n"], int(case["n"] * case["deg"])
    gen = _gen(n * 1009 + case["deg"])
    if case.get("graph", "cl") == "er":
        cdf, perm = None, None
    else:                    # expected degrees ~ i^(-1/1.1), capped at sqrt(sum); vertex ids shuffled
        shape = torch.arange(1, n + 1, dtype=torch.float64, device="cuda") ** (-1.0 / 1.1)
        cap, lo, hi = min(math.sqrt(want), n - 1.0), 0.0, want * 64.0
        for _ in range(60):
            mid = 0.5 * (lo + hi)
            if float(torch.clamp(mid * shape, max=cap).sum()) < want:
                lo = mid
            else:
                hi = mid
        cdf = torch.cumsum(torch.clamp(hi * shape, max=cap), 0)
        cdf = cdf / cdf[-1].item()
        perm = torch.randperm(n, generator=gen, device="cuda")

    def ends(k):
        if cdf is None:
            return torch.randint(n, (k,), generator=gen, device="cuda")
        u = torch.rand(k, generator=gen, device="cuda", dtype=torch.float64)
        return perm[torch.searchsorted(cdf, u).clamp_(max=n - 1)]

    keys = torch.zeros(0, dtype=torch.int64, device="cuda")
    for _ in range(6):       # repeated pairs are dropped and made up for
        missing = want - keys.numel()
        if missing <= want // 100:
            break
        a, b = ends(missing // 2 + 8), ends(missing // 2 + 8)
        ok = a != b
        a, b = a[ok], b[ok]
        keys = torch.unique(torch.cat([keys, a * n + b, b * n + a]))
    if self_loops:
        i = torch.arange(n, device="cuda")
        keys = torch.unique(torch.cat([keys, i * n + i]))
    return keys, gen


def _own_vertices(case, gen, G):
    """A partition's own vertices: frac * n of them grown breadth-first from a random vertex."""
    n, k = G.n_rows, max(1, int(case["n"] * case["frac"]))
    if case.get("graph") == "er":
        return torch.arange(k, device="cuda")
    start = torch.randint(n, (64,), generator=gen, device="cuda")
    length = (G.row_ptr[1:] - G.row_ptr[:-1])[start]
    root = start[torch.argmax((length > 0).int())].int().reshape(1)       # one that has neighbours
    _, ring, _, hop = P.gnn_build_active_sets(G, root, 8, gt=G)
    grown = ring[: min(k, int(hop[-1]))].long()
    mark = torch.zeros(n, dtype=torch.bool, device="cuda")
    mark[grown] = True
    rest = torch.nonzero(~mark).reshape(-1)[: k - grown.numel()]          # a small component: made up with other vertices
    return torch.cat([grown, rest])


def _global_graph(case, gen, self_loops=False):
    """-> the unpartitioned graph and the partition's own vertices, ids ascending."""
    n = case["n"]
    keys, fixed = _structure(case, self_loops)
    own = _own_vertices(case, fixed, _csr(keys, n))
    name = torch.randperm(n, generator=gen, device="cuda")
    keys = torch.sort(name[keys // n] * n + name[keys % n]).values
    return _csr(keys, n), torch.sort(name[own]).values.int()


def _partition(case, gen, hops, self_loops=False):
    """-> local graph numbered by (distance, id), ring offsets, degrees in the unpartitioned graph."""
    G, T = _global_graph(case, gen, self_loops)
    dist, ring, _, hop = P.gnn_build_active_sets(G, T, hops, gt=G)
    local, _ = P.gnn_extract_partition(G, ring, int(hop[-1]), dist, hops)
    degree = (G.row_ptr[1:] - G.row_ptr[:-1])[ring[: int(hop[-1])].long()].contiguous()
    return local, [int(h) for h in hop], degree


def _matrix(gen, n, width, dtype, scale=1.0, relu=False):
    """[n, row_stride(width)] with N(0, scale^2) values (ReLU applied to activations); the pad is zero."""
    m = torch.zeros(n, P.row_stride(width, dtype), dtype=dtype, device="cuda")
    step = max(1, (1 << 27) // width)
    for i in range(0, n, step):
        x = torch.randn(min(step, n - i), width, generator=gen, device="cuda") * scale
        m[i: i + step, :width] = (torch.relu(x) if relu else x).to(dtype)
    return m


def _weights(gen, K, N, dtype):
    return (torch.randn(K, N, generator=gen, device="cuda") / math.sqrt(K)).to(dtype)


def _out(n, width, dtype):
    return torch.zeros(n, P.row_stride(width, dtype), dtype=dtype, device="cuda")


def _scales(case, graph, degree):
    """(row scale, column scale) of a layer's aggregation."""
    if case["model"] == "gcn":
        s = P.gnn_norm_scales(P.GNN_NORM_SYM, graph.n_rows, length=degree)
        return s, s
    return P.gnn_norm_scales(P.GNN_NORM_MEAN, graph.n_rows, row_ptr=graph.row_ptr), None


def prepare(case, seed):
    gen = _gen(seed)
    kind = case["kind"]
    S = {"case": dict(case)}
    dtype = DTYPES[case.get("dtype", "f32")]
    if kind == "step":
        dims = [int(d) for d in case["dims"].split("-")]
        gcn = case["model"] == "gcn"
        graph, hop, degree = _partition(case, gen, len(dims) - 1, self_loops=gcn)
        params = []
        for K, N in zip(dims[:-1], dims[1:]):
            p = {"W_neigh": _weights(gen, K, N, dtype), "bias": 0.1 * torch.randn(N, generator=gen, device="cuda")}
            if not gcn:
                p["W_self"] = _weights(gen, K, N, dtype)
            params.append(p)
        targets = torch.arange(hop[1], dtype=torch.int32, device="cuda")
        model = P.MaskedGNN(graph, graph, targets, case["model"], params, dtype=dtype, global_degree=degree if gcn else None,
                            prefix_numbered=True)
        x = _matrix(gen, graph.n_rows, dims[0], dtype)
        model.set_input(x)
        labels = torch.randint(dims[-1], (hop[1],), generator=gen, device="cuda").int()
        S.update(model=model, labels=labels, dims=dims, hop=hop, graph=graph, params=params, x=x, degree=degree)
    elif kind == "agg":
        graph, hop, degree = _partition(case, gen, case["hops"], self_loops=case["model"] == "gcn")
        rs, cs = _scales(case, graph, degree)
        n, F = graph.n_rows, case["F"]
        fwd = case["dir"] == "fwd"
        # rows of the first layer; backward: the rows of the layer below, gathered from the gradients of those rows
        x = _matrix(gen, n, F, dtype, relu=fwd) if fwd else _matrix(gen, n, F, dtype, scale=1e-3)
        S.update(graph=graph, hop=hop, x=x, y=_out(n, F, dtype), rs=rs, cs=cs, ws=P.Workspace())
        if not fwd:
            S["h"] = _matrix(gen, n, F, dtype, relu=True)
    elif kind == "linear":
        M, K, N = case["M"], case["K"], case["N"]
        up = max(M, int(M * case["up"]))         # rows of the layer below, all of which get an input gradient
        two = case["src"] == 2
        S.update(Wn=_weights(gen, K, N, dtype), Ws=_weights(gen, K, N, dtype) if two else None, ws=P.Workspace(), up=up,
                 a=_matrix(gen, M, K, dtype, scale=0.3), h=_matrix(gen, up, K, dtype, relu=True))
        if case["dir"] == "fwd":
            S.update(bias=0.1 * torch.randn(N, generator=gen, device="cuda"), out=_out(M, N, dtype))
        else:
            S.update(dz=_matrix(gen, up, N, dtype, scale=1e-3), dg=_matrix(gen, up, N, dtype, scale=1e-3), dx=_out(up, K, dtype),
                     dWn=torch.zeros(K, N, device="cuda"), dWs=torch.zeros(K, N, device="cuda") if two else None,
                     db=torch.zeros(N, device="cuda"))
    elif kind == "norm":
        M, F = int(case["M"] * case["up"]), case["F"]
        S.update(M=M, n_res=case["M"], x=_matrix(gen, M, F, dtype), t=_out(M, F, dtype), kept=_out(M, F, dtype), dy=_matrix(gen, M, F, dtype, scale=1e-3),
                 res=_matrix(gen, M, F, dtype, scale=1e-3), dx=_out(M, F, dtype), ws=P.Workspace(),
                 gamma=1.0 + 0.1 * torch.randn(F, generator=gen, device="cuda"), beta=0.1 * torch.randn(F, generator=gen, device="cuda"),
                 dgamma=torch.zeros(F, device="cuda"), dbeta=torch.zeros(F, device="cuda"))
        # the forward output that the backward pass reads: made here, so that a unit that is zero to within rounding is open or
        # closed alike for every implementation of the backward pass
        for i in range(0, M, 1 << 18):
            x = S["x"][i: i + (1 << 18), :F].float()
            x = torch.nn.functional.layer_norm(x, (F,), S["gamma"], S["beta"], 1e-5)
            S["kept"][i: i + (1 << 18), :F] = torch.relu(x).to(dtype)
    elif kind == "mask":
        graph, hop, _ = _partition(case, gen, case["hops"])
        S.update(graph=graph, hop=hop, seed=int(seed) * 7919 + 1)
    else:
        G, T = _global_graph(case, gen)
        S.update(graph=G, targets=T, ws=P.Workspace(), seed=int(seed) * 7919 + 1)
        if kind == "sample":     # how many vertices are reached depends on the sampling seed: kept in buffers with room for all
            S["bits"] = P.gnn_make_bitmap(T, G.n_rows)
            S["l2g"], S["row_ptr"] = (torch.zeros(G.n_rows + 1, dtype=torch.int32, device="cuda") for _ in range(2))
    return S


# ---- one pass -------------------------------------------------------------------------------------------------
def run(S):
    case = S["case"]
    kind = case["kind"]
    if kind == "step":
        m = S["model"]
        loss = m.step(S["labels"])
        return {"loss": loss, "logits": m.H[m.L][: S["hop"][1], : S["dims"][-1]], "grads": m.grads}
    if kind == "agg":
        n_rows = S["hop"][-2]                    # rows of the first layer: all but the outermost ring
        if case["dir"] == "fwd":
            P.gnn_masked_spmm_fwd(S["graph"], None, n_rows, S["x"], S["y"], case["F"], S["rs"], S["cs"], ws=S["ws"])
            return S["y"][:n_rows, : case["F"]]
        n = S["graph"].n_rows
        P.gnn_masked_spmm_bwd(S["graph"], None, n, None, 0, S["x"], S["y"], case["F"], S["rs"], S["cs"], accumulate=False, ws=S["ws"],
                              relu_H=S["h"], src_prefix=n_rows if n_rows < n else -1)
        return S["y"][:, : case["F"]]
    if kind == "linear":
        M, K, N, two = case["M"], case["K"], case["N"], case["src"] == 2
        if case["dir"] == "fwd":
            P.gnn_linear_fwd(None, M, S["a"], S["h"] if two else None, K, S["Wn"], S["Ws"], S["bias"], S["out"], relu=True, ws=S["ws"])
            return S["out"][:, :N]
        P.gnn_linear_bwd(None, M, S["dz"], None, False, S["a"], S["h"] if two else None, K, S["Wn"], S["Ws"], S["dWn"], S["dWs"], S["db"],
                         None, None, ws=S["ws"])
        if two:
            P.gnn_linear_bwd_input2(None, S["up"], S["dg"], S["Wn"], S["dz"], S["Ws"], M, N, K, S["h"], S["dx"], ws=S["ws"])
        else:
            P.gnn_linear_bwd_input(None, S["up"], S["dg"], N, S["Wn"], K, 0, S["h"], S["dx"], ws=S["ws"])
        return {"dWn": S["dWn"], "dWs": S["dWs"], "db": S["db"], "dx": S["dx"][:, :K]}
    if kind == "norm":
        M, F = S["M"], case["F"]
        P.gnn_layer_norm_relu_fwd(None, M, S["x"], F, S["gamma"], S["beta"], S["t"])
        P.gnn_layer_norm_relu_bwd(None, M, S["dy"], S["kept"], S["x"], F, S["gamma"], S["res"], S["n_res"], S["dx"], S["dgamma"], S["dbeta"],
                                  ws=S["ws"])
        return {"t": S["t"][:, :F], "dx": S["dx"][:, :F], "dgamma": S["dgamma"], "dbeta": S["dbeta"]}
    if kind == "extract":
        G = S["graph"]
        dist, ring, off, hop = P.gnn_build_active_sets(G, S["targets"], case["hops"], ws=S["ws"], gt=G)
        local, new_id = P.gnn_extract_partition(G, ring, int(hop[-1]), dist, case["hops"], ws=S["ws"])
        return {"dist": dist, "ring": ring[: int(hop[-1])], "off": off, "row_ptr": local.row_ptr, "col_idx": local.col_idx, "new_id": new_id}
    if kind == "sample":
        G = S["graph"]
        rp, ci = P.gnn_sample_boundary(G, S["bits"], S["targets"], case["fanout"], S["seed"], ws=S["ws"])
        local, l2g, hop = P.gnn_extract_sampled_partition(G, S["targets"], rp, ci, ws=S["ws"])
        S["l2g"][: l2g.numel()].copy_(l2g)
        S["row_ptr"][: l2g.numel() + 1].copy_(local.row_ptr)
        return {"kept_ptr": rp, "kept": ci, "row_ptr": S["row_ptr"], "col_idx": local.col_idx, "l2g": S["l2g"]}
    g = S["graph"]
    if case["rule"] == "fanout":
        how = {"fanout": case["fanout"]}
    else:
        how = {"threshold": (1 << 64) // case["fanout"] - 1}
    keep, kept_len, thr_k, thr_u = P.gnn_layer_edge_mask(g, None, S["hop"][-2], case["rule"], 1, S["seed"], with_thresholds=True, **how)
    keep_t = P.gnn_layer_edge_mask_transposed(g, thr_k, thr_u, 1, S["seed"])
    return {"keep": keep, "kept_len": kept_len, "thr_k": thr_k, "thr_u": thr_u, "keep_t": keep_t}


# ---- what a pass cannot do without ----------------------------------------------------------------------------
def _reached(case, hops):
    """Vertices within so many hops of the partition's own, as a share of all: on these graphs nearly all after two."""
    own = case["frac"]
    return min(1.0, own + (1.0 - own) * (1.0 - math.exp(-own * case["deg"] * hops)))


def work(case):
    kind = case["kind"]
    es = 4 if case.get("dtype", "f32") == "f32" else 2
    if kind == "step":
        dims = [int(d) for d in case["dims"].split("-")]
        L = len(dims) - 1
        rows = [case["n"] * _reached(case, L - l) if l < L else case["n"] * case["frac"] for l in range(L + 1)]
        nbytes, flops, src = 0.0, 0.0, 2 if case["model"] == "sage" else 1
        for l in range(1, L + 1):
            K, N = dims[l - 1], dims[l]
            edges = rows[l] * case["deg"]
            passes = 1 if l == 1 else 2          # forward and, but for the first layer, backward
            nbytes += passes * (4.0 * edges + es * (rows[l - 1] * K + rows[l] * N)) + es * rows[l] * (K + N)
            flops += passes * 2.0 * edges * min(K, N) + (1 + passes) * 2.0 * src * rows[l] * K * N
        return {"bytes": nbytes, "flops": flops}
    if kind == "agg":
        n, F = case["n"] * _reached(case, case["hops"]), case["F"]
        rows = case["n"] * _reached(case, case["hops"] - 1) if case["hops"] > 1 else case["n"] * case["frac"]
        edges = rows * case["deg"]
        extra = es * n * F if case["dir"] == "bwd" else 0.0          # the activations of the ReLU
        return {"bytes": 4.0 * edges + es * F * (n + rows) + 8.0 * n + extra, "flops": 2.0 * edges * F}
    if kind == "linear":
        M, K, N, src, up = case["M"], case["K"], case["N"], case["src"], case["M"] * case["up"]
        w = es * src * K * N
        if case["dir"] == "fwd":
            return {"bytes": es * M * (src * K + N) + w, "flops": 2.0 * src * M * K * N}
        return {"bytes": es * (M * (K + N) + up * (2 * K + N)) + w + 4.0 * src * K * N,
                "flops": 2.0 * src * M * K * N + 2.0 * K * N * (up + (src - 1) * M)}
    if kind == "norm":
        M, F = case["M"] * case["up"], case["F"]
        return {"bytes": es * M * F * 4.0 + es * case["M"] * F, "flops": 20.0 * M * F}
    if kind == "extract":
        n = case["n"] * _reached(case, case["hops"])
        return {"bytes": 8.0 * n * case["deg"] + 20.0 * case["n"], "flops": 0.0}
    if kind == "sample":
        own = case["n"] * case["frac"]
        kept = own * min(case["deg"], case["fanout"] + case["deg"] * case["frac"])
        return {"bytes": 4.0 * own * case["deg"] + 16.0 * kept + 16.0 * case["n"], "flops": 0.0}
    edges = case["n"] * _reached(case, case["hops"]) * case["deg"]
    return {"bytes": 2.0 * (4.0 + 0.125) * edges + 16.0 * case["n"], "flops": 0.0}


def tolerance(case):
    if case["kind"] in ("extract", "sample", "mask"):
        return "exact"
    if case["kind"] == "step":
        return {"rel": 3e-3, "max": 2e-1}        # a unit of a ReLU that is zero to within rounding passes its gradient or not
    if case.get("dtype") == "bf16":
        return {"rel": 7e-3, "max": 2e-2}
    return {"rel": 2e-6, "max": 8e-5}


# ---- the same in 64 bits --------------------------------------------------------------------------------------
def _aggregate64(graph, n_rows, x, rs, cs, limit=None):
    """rs * sum over the row of cs * x, for the rows 0 .. n_rows-1; only the neighbours below `limit`."""
    x = x if cs is None else x * cs.double()[: x.shape[0], None]
    if limit is not None and limit < x.shape[0]:
        x = x.clone()
        x[limit:] = 0.0
    F = x.shape[1]
    row_ptr = graph.row_ptr.long()
    ends = row_ptr[: n_rows + 1].cpu()
    out = torch.zeros(n_rows, F, dtype=torch.float64, device="cuda")
    most, r0 = max(1, (1 << 31) // max(F, 1)), 0
    while r0 < n_rows:
        r1 = int(torch.searchsorted(ends, ends[r0] + most, right=True)) - 1
        r1 = min(n_rows, max(r1, r0 + 1))
        e0, e1 = int(ends[r0]), int(ends[r1])
        if e1 > e0:
            out[r0:r1] = torch.segment_reduce(x[graph.col_idx[e0:e1].long()], "sum", offsets=row_ptr[r0: r1 + 1] - e0, axis=0, initial=0.0)
        r0 = r1
    return out if rs is None else out * rs.double()[:n_rows, None]


def _exact_step(S):
    case, graph, hop, dims, params = S["case"], S["graph"], S["hop"], S["dims"], S["params"]
    L, gcn = len(dims) - 1, case["model"] == "gcn"
    if gcn:
        rs = cs = S["degree"].double().rsqrt()
    else:
        length = (graph.row_ptr[1:] - graph.row_ptr[:-1]).double()
        rs, cs = torch.where(length > 0, 1.0 / length, torch.zeros_like(length)), None
    rows = [hop[L - l + 1] for l in range(L + 1)]
    W = [{k: v.double() for k, v in p.items()} for p in params]
    H, A = [S["x"][:, : dims[0]].double()], [None]
    for l in range(1, L + 1):
        a = _aggregate64(graph, rows[l], H[l - 1], rs, cs)
        z = a @ W[l - 1]["W_neigh"] + W[l - 1]["bias"]
        if not gcn:
            z = z + H[l - 1][: rows[l]] @ W[l - 1]["W_self"]
        A.append(a)
        H.append(torch.relu(z) if l < L else z)
    y = S["labels"].long()
    loss = torch.nn.functional.cross_entropy(H[L], y)
    d = torch.softmax(H[L], 1)
    d[torch.arange(d.shape[0], device="cuda"), y] -= 1.0
    d = d / d.shape[0]
    grads = [None] * L
    for l in range(L, 0, -1):
        g = {"dW_neigh": A[l].T @ d, "dbias": d.sum(0)}
        if not gcn:
            g["dW_self"] = H[l - 1][: rows[l]].T @ d
        grads[l - 1] = g
        if l > 1:
            da = torch.zeros(graph.n_rows, dims[l - 1], dtype=torch.float64, device="cuda")
            da[: rows[l]] = d @ W[l - 1]["W_neigh"].T
            dx = _aggregate64(graph, rows[l - 1], da, cs, rs)
            if not gcn:
                dx[: rows[l]] += d @ W[l - 1]["W_self"].T
            d = torch.where(H[l - 1] > 0, dx, torch.zeros_like(dx))
    # below the last layer a gradient passes a ReLU whose input may be zero to within rounding, on either side: the few units
    # for which 32 and 64 bits decide differently make up its whole difference, so there is no value to hold it against
    grads[:-1] = [{k: None for k in g} for g in grads[:-1]]
    return {"loss": loss.reshape(1), "logits": H[L], "grads": grads}


def exact(case, seed):
    kind = case["kind"]
    if kind in ("extract", "sample", "mask"):
        return None
    S = prepare(case, seed)
    if kind == "step":
        return _exact_step(S)
    if kind == "agg":
        F, n_rows = case["F"], S["hop"][-2]
        x = S["x"][:, :F].double()
        if case["dir"] == "fwd":
            return _aggregate64(S["graph"], n_rows, x, S["rs"], S["cs"])
        out = _aggregate64(S["graph"], S["graph"].n_rows, x, S["cs"], S["rs"], limit=n_rows)
        return torch.where(S["h"][:, :F] > 0, out, torch.zeros_like(out))
    if kind == "linear":
        M, K, N, two = case["M"], case["K"], case["N"], case["src"] == 2
        a, h, Wn = S["a"][:, :K].double(), S["h"][:, :K].double(), S["Wn"].double()
        Ws = S["Ws"].double() if two else None
        if case["dir"] == "fwd":
            z = a @ Wn + S["bias"].double()
            return torch.relu(z + h[:M] @ Ws if two else z)
        dz, dg = S["dz"][:, :N].double(), S["dg"][:, :N].double()
        dx = dg @ Wn.T
        if two:
            dx[:M] += dz[:M] @ Ws.T
        return {"dWn": a.T @ dz[:M], "dWs": h[:M].T @ dz[:M] if two else None, "db": dz[:M].sum(0),
                "dx": torch.where(h > 0, dx, torch.zeros_like(dx))}
    F = case["F"]
    x, dy, gamma, beta = S["x"][:, :F].double(), S["dy"][:, :F].double(), S["gamma"].double(), S["beta"].double()
    dev = x - x.mean(1, keepdim=True)
    rstd = torch.rsqrt((dev * dev).mean(1, keepdim=True) + 1e-5)
    xh = dev * rstd
    t = torch.relu(xh * gamma + beta)
    g = torch.where(S["kept"][:, :F] > 0, dy, torch.zeros_like(dy))
    gg = g * gamma
    dx = rstd * (gg - gg.mean(1, keepdim=True) - xh * (gg * xh).mean(1, keepdim=True))
    dx[: S["n_res"]] += S["res"][: S["n_res"], :F].double()
    return {"t": t, "dx": dx, "dgamma": (g * xh).sum(0), "dbeta": g.sum(0)}
