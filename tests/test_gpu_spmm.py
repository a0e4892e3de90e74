"""GPU parity: gnn_masked_spmm_fwd / _bwd against the oracle (section 2.1 aggregation under
the section 6 mask).  fp32: 1e-4, bf16 storage: 2e-2 (see gpu_util.TOL)."""
import numpy as np
import pytest
import torch

import graphgen as gg
import oracle
from gpu_util import as_stored, check, dev, host64, padded

pytestmark = pytest.mark.gpu

SENTINEL = 12345.0


def _used_blocked_route(ws):
    """The size query reports 0 bytes when the column-blocked route does not apply, so the workspace stays minimal."""
    return ws is not None and ws.buf is not None and ws.buf.numel() > 256


def _fwd_case(g, F, ld, dtype, rows, scales, seed, ws=None):
    import paper_2311_06837_amd as P
    print(f"spmm fwd: n={g.n_rows} nnz={g.nnz} F={F} ld={ld} {dtype} rows={'list' if rows is not None else 'all'} "
          f"scales={scales}", flush=True)
    rng = np.random.default_rng(seed)
    n = g.n_rows
    X = as_stored(rng.standard_normal((n, F)), dtype)
    rs = (rng.random(n) + 0.5).astype(np.float32) if scales else None
    cs = (rng.random(n) + 0.5).astype(np.float32) if scales else None
    G = P.Graph.from_numpy(g.row_ptr, g.col_idx)
    Xd = padded(X, ld, dtype, fill=float("nan") if ld > F else 0.0)       # pad columns must never matter
    if ld > F and ld - F >= 1:
        Xd[:, F:] = float("nan")
    Yd = torch.full((n, ld), SENTINEL, dtype=dtype, device="cuda")
    rows_d = dev(rows) if rows is not None else None
    n_active = len(rows) if rows is not None else n
    P.gnn_masked_spmm_fwd(G, rows_d, n_active, Xd, Yd, F, dev(rs) if scales else None, dev(cs) if scales else None, ws=ws)
    torch.cuda.synchronize()
    want = np.full((n, F), SENTINEL)
    oracle.spmm_fwd(g.row_ptr, g.col_idx, rows, X, want, F, rs, cs)
    got = host64(Yd)
    sel = np.asarray(rows if rows is not None else np.arange(n))
    check(got[sel, :F], want[sel], dtype, "active rows")
    rest = np.setdiff1d(np.arange(n), sel)
    assert (got[rest] == host64(torch.tensor(SENTINEL, dtype=dtype))).all(), "masked rows were written"
    if ld > F:
        assert (got[:, F:] == host64(torch.tensor(SENTINEL, dtype=dtype))).all(), "pad columns were written"


def _fwd_add_case(g, F, ld, dtype, rows, relu, seed, ws=None, bias=False):
    """gnn_masked_spmm_fwd_add: Y = act(Y + aggregation).  The oracle aggregates into a zeroed matrix; the sum with
    the self term and the ReLU are written out here (in the storage precision of the self term).  bias: the form
    without a self term - the listed rows start from a bias vector, whatever the output matrix held."""
    import paper_2311_06837_amd as P
    print(f"spmm fwd_add: n={g.n_rows} nnz={g.nnz} F={F} ld={ld} {dtype} rows={'list' if rows is not None else 'all'} relu={relu}",
          flush=True)
    rng = np.random.default_rng(seed)
    n = g.n_rows
    X = as_stored(rng.standard_normal((n, F)), dtype)
    S = as_stored(rng.standard_normal((n, F)), dtype)
    rs = (1.0 / np.maximum(g.degrees(), 1)).astype(np.float32)
    G = P.Graph.from_numpy(g.row_ptr, g.col_idx)
    Xd = padded(X, ld, dtype)
    Yd = torch.full((n, ld), SENTINEL, dtype=dtype, device="cuda")
    Yd[:, :F] = padded(S, F, dtype)
    rows_d = dev(rows) if rows is not None else None
    n_active = len(rows) if rows is not None else n
    b = (rng.standard_normal(F) * 0.5).astype(np.float32) if bias else None
    P.gnn_masked_spmm_fwd_add(G, rows_d, n_active, Xd, Yd, F, dev(rs), None, relu=relu, ws=ws, bias=dev(b) if bias else None)
    torch.cuda.synchronize()
    agg = np.zeros((n, F))
    oracle.spmm_fwd(g.row_ptr, g.col_idx, rows, X, agg, F, rs, None)
    start = np.broadcast_to(as_stored(b.astype(np.float64), dtype), (n, F)) if bias else S
    want = start + agg
    if relu:
        want = np.maximum(want, 0.0)
    got = host64(Yd)
    sel = np.asarray(rows if rows is not None else np.arange(n))
    check(got[sel, :F], want[sel], dtype, "active rows")
    if relu:
        assert (got[sel, :F] >= 0).all()
        # a row without neighbours still gets its activation
        empty = sel[g.degrees()[sel] == 0]
        assert np.array_equal(got[empty, :F], np.maximum(start[empty], 0.0))
    rest = np.setdiff1d(np.arange(n), sel)
    assert np.array_equal(got[rest, :F], S[rest]), "masked rows were written"
    if ld > F:
        assert (got[:, F:] == host64(torch.tensor(SENTINEL, dtype=dtype))).all(), "pad columns were written"


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("relu", [False, True])
def test_fwd_add_on_top_of_the_self_term(dtype, relu):
    g = gg.chung_lu(3000, 6.0, 2.1, 13)
    assert (g.degrees() == 0).any()
    rng = np.random.default_rng(3)
    rows = np.sort(rng.choice(3000, 1777, replace=False)).astype(np.int32)
    _fwd_add_case(g, 256, 256, dtype, None, relu, 51)
    _fwd_add_case(g, 100, 104, dtype, rows, relu, 52)
    _fwd_add_case(g, 7, 7, dtype, rows, relu, 53)            # element-wise lanes
    _fwd_add_case(g, 16, 16, dtype, rows, relu, 54)          # narrow rows
    _fwd_add_case(g, 41, 48, dtype, None, relu, 55)
    _fwd_add_case(g, 47, 48, dtype, rows, relu, 56, bias=True)     # no self term: the rows start from the bias
    _fwd_add_case(g, 256, 256, dtype, None, relu, 57, bias=True)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("F,ld", [(64, 64), (100, 100), (128, 128), (256, 256), (602, 608), (602, 602), (7, 7), (1, 8),
                                  (300, 304), (1000, 1000), (16, 16), (32, 32), (41, 44), (47, 48)])
def test_fwd_widths(dtype, F, ld):
    g = gg.chung_lu(3000, 20.0, 2.1, 11)
    rng = np.random.default_rng(F)
    rows = np.sort(rng.choice(3000, 1777, replace=False)).astype(np.int32)
    _fwd_case(g, F, ld, dtype, rows, True, F)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_fwd_hub_rows_empty_rows_and_all_rows(dtype):
    g = gg.chung_lu(12000, 150.0, 2.1, 12)                                # hub rows > 1024 neighbours
    assert g.degrees().max() > 1024
    _fwd_case(g, 128, 128, dtype, None, True, 1)
    _fwd_case(g, 602, 608, dtype, None, False, 2)
    d = gg.random_directed(5000, 1.5, 13)                                 # many empty rows
    assert (d.degrees() == 0).any()
    _fwd_case(d, 64, 64, dtype, None, True, 3)
    rows = np.random.default_rng(0).permutation(5000)[:3001].astype(np.int32)     # unsorted row list, ragged count
    _fwd_case(d, 100, 100, dtype, rows, False, 4)


def test_fwd_sum_of_ones_is_degree_exactly():
    import paper_2311_06837_amd as P
    g = gg.chung_lu(20000, 80.0, 2.1, 14)
    G = P.Graph.from_numpy(g.row_ptr, g.col_idx)
    X = torch.ones(20000, 64, device="cuda")
    Y = torch.zeros(20000, 64, device="cuda")
    P.gnn_masked_spmm_fwd(G, None, 20000, X, Y, 64)
    assert torch.equal(Y[:, 0].cpu(), torch.from_numpy(g.degrees()).float())     # integers < 2^24 are exact in fp32
    assert torch.equal(Y, Y[:, :1].expand(-1, 64))


def test_fwd_is_bitwise_reproducible():
    import paper_2311_06837_amd as P
    g = gg.chung_lu(12000, 150.0, 2.1, 12)
    G = P.Graph.from_numpy(g.row_ptr, g.col_idx)
    X = torch.randn(12000, 256, device="cuda", generator=torch.Generator("cuda").manual_seed(0))
    outs = []
    for _ in range(3):
        Y = torch.zeros(12000, 256, device="cuda")
        P.gnn_masked_spmm_fwd(G, None, 12000, X, Y, 256)
        outs.append(Y)
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])


def _bwd_case(g, F, ld, dtype, L, lyr, accumulate, seed, ws=None, relu=False):
    """Backward of layer `lyr` of an L-layer model: forward rows R_lyr, outputs for R_{lyr-1}.  relu: the call also
    undoes the ReLU of the layer in front (what it stores is zeroed where that layer's activations are <= 0)."""
    import paper_2311_06837_amd as P
    print(f"spmm bwd: n={g.n_rows} nnz={g.nnz} F={F} ld={ld} {dtype} L={L} layer={lyr} acc={accumulate} relu={relu}", flush=True)
    rng = np.random.default_rng(seed)
    n = g.n_rows
    T = np.sort(rng.choice(n, max(1, n // 50), replace=False)).astype(np.int32)
    dist, ring, off = oracle.active_sets(g.row_ptr, g.col_idx, T, L)
    rows_f = ring[: off[L - lyr + 1]]                 # R_lyr
    rows_o = ring[: off[L - lyr + 2]]                 # R_{lyr-1}
    gt = gg.transpose(g)
    dY = as_stored(rng.standard_normal((n, F)), dtype)
    rs = (rng.random(n) + 0.5).astype(np.float32)
    cs = (rng.random(n) + 0.5).astype(np.float32)
    init = as_stored(rng.standard_normal((n, F)), dtype) if accumulate else np.full((n, F), SENTINEL)
    GT = P.Graph.from_numpy(gt.row_ptr, gt.col_idx)
    dYd = padded(dY, ld, dtype)
    dXd = padded(init, ld, dtype, fill=SENTINEL)
    Hact = as_stored(np.maximum(rng.standard_normal((n, F)), 0), dtype) if relu else None     # about half of it is zero
    P.gnn_masked_spmm_bwd(GT, dev(rows_o), len(rows_o), dev(dist), L - lyr, dYd, dXd, F, dev(rs), dev(cs), accumulate=accumulate,
                          ws=ws, relu_H=padded(Hact, ld, dtype, fill=float("nan") if ld > F else 0.0) if relu else None)
    torch.cuda.synchronize()
    want = np.zeros((n, F))
    oracle.spmm_bwd(g.row_ptr, g.col_idx, rows_f, dY, want, F, rs, cs)
    # everything the adjoint touches lies inside R_{lyr-1}
    outside = np.setdiff1d(np.arange(n), rows_o)
    assert not want[outside].any()
    if accumulate:
        want = want + init
    if relu:
        want = want * (Hact > 0)
    got = host64(dXd)
    check(got[rows_o, :F], want[rows_o], dtype, "bwd rows")
    assert (got[outside, :F] == host64(padded(init, ld, dtype, fill=SENTINEL))[outside, :F]).all(), "rows outside were written"


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("accumulate", [False, True])
def test_bwd_directed_graph_with_filter(dtype, accumulate):
    g = gg.random_directed(8000, 6.0, 21)
    _bwd_case(g, 128, 128, dtype, 3, 3, accumulate, 5)
    _bwd_case(g, 256, 256, dtype, 3, 2, accumulate, 6)
    _bwd_case(g, 602, 608, dtype, 2, 2, accumulate, 7)
    _bwd_case(g, 16, 16, dtype, 3, 2, accumulate, 8)                     # narrow rows: 4 / 8 lanes per row
    _bwd_case(g, 41, 48, dtype, 3, 3, accumulate, 9)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("accumulate", [False, True])
def test_bwd_that_undoes_the_relu_in_front(dtype, accumulate):
    g = gg.random_directed(8000, 6.0, 22)
    _bwd_case(g, 128, 128, dtype, 3, 3, accumulate, 15, relu=True)
    _bwd_case(g, 602, 608, dtype, 2, 2, accumulate, 16, relu=True)
    _bwd_case(g, 100, 100, dtype, 2, 2, accumulate, 17, relu=True)       # unaligned for bf16: element route
    _bwd_case(g, 7, 7, dtype, 2, 2, accumulate, 18, relu=True)
    h = gg.chung_lu(12000, 150.0, 2.1, 12)                                # hub rows: reduced through LDS, then masked
    _bwd_case(h, 64, 64, dtype, 2, 2, accumulate, 19, relu=True)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_bwd_power_law_hubs(dtype):
    g = gg.chung_lu(12000, 150.0, 2.1, 12)
    _bwd_case(g, 64, 64, dtype, 2, 2, False, 8)
    _bwd_case(g, 100, 100, dtype, 3, 2, True, 9)
    _bwd_case(g, 16, 16, dtype, 2, 2, True, 10, relu=True)               # hub rows reduced by 64 narrow lane groups
    _bwd_case(g, 32, 32, dtype, 2, 2, False, 11)


def test_empty_calls_are_noops():
    import paper_2311_06837_amd as P
    g = gg.erdos_renyi(100, 3.0, 1)
    G = P.Graph.from_numpy(g.row_ptr, g.col_idx)
    with pytest.raises(P.GnnError):             # a source prefix is -1 (none) or a vertex count
        z = torch.zeros(100, 8, device="cuda")
        P.gnn_masked_spmm_bwd(G, None, 100, None, 0, z, torch.zeros_like(z), 8, src_prefix=-2)
    X = torch.randn(100, 8, device="cuda")
    Y = torch.full((100, 8), 3.0, device="cuda")
    P.gnn_masked_spmm_fwd(G, None, 0, X, Y, 8)
    P.gnn_masked_spmm_fwd(G, None, 100, X, Y, 0)
    torch.cuda.synchronize()
    assert (Y == 3.0).all()


# ---- column-blocked route (dense graph + workspace) ------------------------------------------

_DENSE = {}


def _dense_graph(deg=88.0):
    """70k vertices (a 256-byte feature slab of 17.9 MB), average row length 90 (bfloat16 takes the route from longer rows on), plus one
    vertex adjacent to 20k others, so that one of its column blocks alone is longer than the hub threshold."""
    if deg not in _DENSE:
        n = 70000
        base = gg.erdos_renyi(n, deg, 31)
        rng = np.random.default_rng(32)
        nb = rng.choice(n - 1, 20000, replace=False).astype(np.int64) + 1      # neighbours of vertex 0
        r = np.repeat(np.arange(n, dtype=np.int64), np.diff(base.row_ptr))
        c = base.col_idx.astype(np.int64)
        z = np.zeros_like(nb)
        _DENSE[deg] = gg.csr_from_edges(n, n, np.concatenate([r, z, nb]), np.concatenate([c, nb, z]))
    return _DENSE[deg]


def _dense_enough(dtype):
    return _dense_graph(88.0 if dtype == torch.float32 else 190.0)


def _blocked(case, *args, **kwargs):
    """A case with a workspace of its own, which must have taken the column-blocked route."""
    import paper_2311_06837_amd as P
    ws = P.Workspace()
    case(*args, ws=ws, **kwargs)
    assert _used_blocked_route(ws), (args[1:], kwargs)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_blocked_route_forward(dtype):
    g, f32 = _dense_enough(dtype), dtype == torch.float32
    assert g.nnz / g.n_rows >= 64 and g.degrees()[0] > 8 * 1024
    _blocked(_fwd_case, g, 200, 200, dtype, None, True, 41)               # 7 (fp32) / 4 (bf16) lines, ragged last line
    rows = np.random.default_rng(5).permutation(g.n_rows)[:40001].astype(np.int32)   # unsorted list, ragged count
    if 0 not in rows:
        rows[17] = 0
    _blocked(_fwd_case, g, 602, 608, dtype, rows, False, 42)
    _blocked(_fwd_case, g, 200, 200, dtype, rows, True, 48)
    _blocked(_fwd_case, g, 64 if f32 else 128, 64 if f32 else 128, dtype, rows, f32, 43)       # a single slab


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_blocked_route_forward_add(dtype):
    g, f32 = _dense_enough(dtype), dtype == torch.float32
    _blocked(_fwd_add_case, g, 200, 200, dtype, None, True, 44)
    rows = np.random.default_rng(6).permutation(g.n_rows)[:40001].astype(np.int32)
    _blocked(_fwd_add_case, g, 256, 256, dtype, rows, False, 45)
    _blocked(_fwd_add_case, g, 90, 96, dtype, rows, f32, 46)
    _blocked(_fwd_add_case, g, 200, 200, dtype, rows, True, 47, bias=True)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("accumulate", [False, True])
def test_blocked_route_backward_with_filter(dtype, accumulate):
    g, F = (_dense_graph(), 136) if dtype == torch.float32 else (_dense_graph(205.0), 264)      # a ragged last slab
    _blocked(_bwd_case, g, F, F, dtype, 2, 2, accumulate, 44)            # forward rows = targets only: most neighbours filtered out
    _blocked(_bwd_case, g, F, F, dtype, 2, 2, accumulate, 45, relu=True)  # the plane sum undoes the ReLU in front


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("wide", [False, True])
def test_blocked_route_row_lengths(dtype, wide):
    """Rows without an edge in a block, of one edge, of a stretch and its neighbours, and over several staged pieces, in
    runs of like length; with a gathered matrix below and above 4 GB (its rows far apart)."""
    import paper_2311_06837_amd as P
    n_rows, n_cols, F = 4999, 70_001, 75
    rng = np.random.default_rng(8)
    lens = np.full(n_rows, 130)
    lens[100:400] = 0
    lens[400:700] = 1
    lens[700:1000] = rng.integers(0, 70, 300)
    lens[1000:1003] = [n_cols, 0, n_cols]
    lens[1500:1520] = 9000
    lens[-1] = n_cols
    cols = [np.sort(rng.choice(n_cols, k, replace=False)).astype(np.int32) for k in lens]
    cols[2000] = np.arange(130, dtype=np.int32)                      # all in one block
    lens[2000] = 130
    rp = np.zeros(n_rows + 1, np.int32)
    rp[1:] = np.cumsum(lens)
    G = P.Graph(torch.from_numpy(rp).cuda(), torch.from_numpy(np.concatenate(cols)).cuda(), n_cols=n_cols, sorted_columns=True)
    ld = (1 << 32) // n_cols // dtype.itemsize // 64 * 64 + 64 if wide else 80
    X = torch.empty((n_cols, ld), dtype=dtype, device="cuda")
    assert (X.numel() * dtype.itemsize >= 1 << 32) == wide
    X[:, :F] = torch.from_numpy(rng.standard_normal((n_cols, F)).astype(np.float32)).cuda()
    Y = torch.zeros((n_rows, 80), dtype=dtype, device="cuda")
    ws = P.Workspace()
    P.gnn_masked_spmm_fwd(G, None, n_rows, X, Y, F, ws=ws)
    assert _used_blocked_route(ws) and ws.buf.numel() == _stream_bytes(G, n_rows, F, ld, dtype, False)      # too few rows for the fours
    x = X[:, :F].double().cpu().numpy()
    want = np.stack([x[c].sum(0) for c in cols])
    size = np.stack([np.abs(x[c]).sum(0) for c in cols])
    got = Y[:, :F].double().cpu().numpy()
    # fp32 sums in any order: at most (terms + 8 planes) * 2^-24 of the sum of magnitudes; then bf16 rounding, 2^-8 of the value
    tol = (lens[:, None] + 8) * 2.0 ** -24 * size + (2.0 ** -8 * np.abs(want) if dtype == torch.bfloat16 else 0.0)
    assert (np.abs(got - want) <= tol).all()
    assert not Y[:, F:].any()


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("form", ["few ids hold most entries", "two passes", "dist filter"])
def test_blocked_route_streams(dtype, form):
    """Rows of 0 to 9 entries in a block, rows over all lane groups and several stages, a last row that is not asked for; a block
    whose share of the ids would not fit 16 bits; 16 blocks in two passes; a neighbour scale; infinities and NaN, which
    must reach the rows that name them and no others."""
    import paper_2311_06837_amd as P
    n_cols = 300_001 if form == "two passes" else 262_144
    n_rows, few = 4300, 1000
    F = 27 if dtype == torch.float32 else 59           # a line, which takes the fours from few rows on
    rng = np.random.default_rng(23)
    lens = np.full(n_rows, 560)
    lens[:300] = rng.integers(0, 80, 300)
    lens[300:400] = 0
    lens[1000:1003] = [100_000, 0, 60_000]
    cols = []
    for k in lens:
        c = rng.choice(n_cols, k, replace=False)
        if form == "few ids hold most entries" and k < few:
            c = np.union1d(rng.choice(few, min(k, 500), replace=False), c[: k // 20])
        cols.append(np.sort(c).astype(np.int32))
    lens = np.array([len(c) for c in cols])
    rp = np.zeros(n_rows + 1, np.int32)
    rp[1:] = np.cumsum(lens)
    G = P.Graph(dev(rp), dev(np.concatenate(cols)), n_cols=n_cols, sorted_columns=True)
    x = as_stored(rng.standard_normal((n_cols, F)), dtype)
    x[[5, 77_777, 222_222], [0, F - 1, 3]] = [np.inf, np.nan, -np.inf]
    scale = (rng.random(n_cols) + 0.5).astype(np.float32)
    dist = (np.arange(n_cols) % 3).astype(np.int32) if form == "dist filter" else None
    X, Y = padded(x, 72, dtype), torch.full((n_rows, 72), SENTINEL, dtype=dtype, device="cuda")
    ws = P.Workspace()
    print(form, dtype, int(lens.sum()), flush=True)
    if dist is None:
        P.gnn_masked_spmm_fwd(G, None, n_rows - 1, X, Y, F, None, dev(scale), ws=ws)
    else:
        P.gnn_masked_spmm_bwd(G, None, n_rows - 1, dev(dist), 1, X, Y, F, dev(scale), None, accumulate=False, ws=ws)
        cols = [c[dist[c] <= 1] for c in cols]
    assert _used_blocked_route(ws)
    blocks = 16 if form == "two passes" else 8
    assert ws.buf.numel() != _stream_bytes(G, n_rows - 1, F, 72, dtype, True, dist is not None, blocks)      # the fours, not the stream kernel
    w = x * scale[:, None].astype(np.float64)
    got = host64(Y)
    untouched = host64(torch.full((1,), SENTINEL, dtype=dtype))      # as the type holds it
    assert (got[n_rows - 1:] == untouched).all() and (got[:, F:] == untouched).all()
    for r, c in enumerate(cols[: n_rows - 1]):
        want, size = w[c].sum(0), np.abs(w[c]).sum(0)
        ok = np.isfinite(want)
        # fp32 sums in any order: at most (terms + 8 planes + the scaled factor) * 2^-24 of the sum of magnitudes; then bf16 rounding
        tol = (len(c) + 9) * 2.0 ** -24 * size[ok] + (2.0 ** -8 * np.abs(want[ok]) if dtype == torch.bfloat16 else 0.0)
        assert (np.abs(got[r, :F][ok] - want[ok]) <= tol).all(), r
        assert np.array_equal(got[r, :F][~ok], want[~ok], equal_nan=True), r


def _random_rows(n_rows, n_cols, longest, seed):
    """Rows of 0 to `longest` entries, ascending and distinct; made on the GPU.  -> Graph, row of every entry, columns"""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    lens = torch.randint(longest + 1, (n_rows,), generator=gen, device="cuda")
    lens[17], lens[18], lens[-1] = 0, longest, longest
    row = torch.repeat_interleave(torch.arange(n_rows, device="cuda"), lens)
    keys = torch.unique(row * n_cols + torch.randint(n_cols, row.shape, generator=gen, device="cuda"))
    row, col = keys // n_cols, keys % n_cols
    row_ptr = torch.zeros(n_rows + 1, dtype=torch.int64, device="cuda")
    row_ptr[1:] = torch.cumsum(torch.bincount(row, minlength=n_rows), 0)
    return _graph(row_ptr, col, n_cols), row, col


def _graph(row_ptr, col, n_cols):
    import paper_2311_06837_amd as P
    return P.Graph(row_ptr.int(), col.int(), n_cols=n_cols, sorted_columns=True)


def _check_sums(got, row, col, n_rows, x, scale, dtype):
    """got[0:n_rows] against float64 sums over the entries (row, col): fp32 sums in any order are off by at most (terms + 8 planes +
    the scaled factor) * 2^-24 of the sum of magnitudes; then bf16 rounding, 2^-8 of the value."""
    keep = row < n_rows
    row, col = row[keep], col[keep]
    lens = torch.bincount(row, minlength=n_rows)
    w = x.double() * (1.0 if scale is None else scale.double()[:, None])
    for c0 in range(0, x.shape[1], 64):
        terms = w[:, c0: c0 + 64]
        want = torch.segment_reduce(terms[col], "sum", lengths=lens, axis=0, initial=0.0)
        size = torch.segment_reduce(terms.abs()[col], "sum", lengths=lens, axis=0, initial=0.0)
        tol = (lens[:, None] + 9) * 2.0 ** -24 * size + (2.0 ** -8 * want.abs() if dtype == torch.bfloat16 else 0.0)
        assert ((got[:n_rows, c0: c0 + 64].double() - want).abs() <= tol).all()


def _stream_bytes(G, n_active, F, ld, dtype, scaled, filtered=False, blocks=8):
    """Workspace of the stream kernel's form: cut points, planes, prepared ids (filter) and factors (bf16) or scaled rows (fp32),
    boundaries, samples."""
    up = lambda nbytes: -(-nbytes // 256) * 256
    factors = scaled and dtype == torch.bfloat16
    need = up(n_active * (blocks + 1) * 4) + up(8 * n_active * (-(-F // 8) * 8) * 4) + up((blocks + 1) * 4) + up(131072 * (4 if filtered else 2))
    if filtered or factors:
        need += up(n_active * blocks * 4) + up(G.nnz * 4)
    if factors:
        need += up(G.nnz * 4)
    elif scaled:
        need += up(G.n_cols * ld * 4)
    return need


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("scaled", [False, True])
@pytest.mark.parametrize("F", [256, 60, 40, 24])
def test_blocked_route_copies_rows_only_where_the_call_pays_for_it(F, scaled, dtype):
    """A call over few of the rows takes the stream kernel, which gathers in place, and one over many the fours, which have a copy of
    the gathered rows in the workspace; the sums agree with float64 on either side of the line."""
    import paper_2311_06837_amd as P
    one_line, one_slab = F * dtype.itemsize <= 128, dtype == torch.float32 and F * 4 <= 256
    if dtype == torch.bfloat16 and F < 60:
        pytest.skip("as 60 columns: one line")
    n_cols, longest = 66_000, (400 if dtype == torch.float32 else 1100 if scaled else 900) if one_line else 1100       # half as many on average
    if one_line:
        entries, share = (1e6 if scaled else 2e6), 0.0
    else:
        entries, share = (4e6 if scaled else 6e6), 1 / ((6 if scaled else 3) if one_slab else (16 if scaled else 10))
    at = max(int(entries / (longest / 2)), int(n_cols * share))
    few, many = max(4096, int(0.95 * at)), max(4096, int(1.05 * at))
    G, row, col = _random_rows(int(1.1 * many), n_cols, longest, 5)
    gen = torch.Generator(device="cuda").manual_seed(6)
    ld = P.row_stride(F, dtype)
    X = torch.full((n_cols, ld), float("nan"), dtype=dtype, device="cuda")
    X[:, :F] = torch.randn(n_cols, F, generator=gen, device="cuda").to(dtype)
    scale = torch.rand(n_cols, generator=gen, device="cuda") + 0.5 if scaled else None
    for n_active in (few, many):
        Y = torch.full((G.n_rows, ld), SENTINEL, dtype=dtype, device="cuda")
        ws = P.Workspace()
        P.gnn_masked_spmm_fwd(G, None, n_active, X, Y, F, None, scale, ws=ws)
        more = ws.buf.numel() - _stream_bytes(G, n_active, F, ld, dtype, scaled)
        print(n_active, F, dtype, scaled, ws.buf.numel(), more, flush=True)
        if n_active == few < many:
            assert more == 0
        else:      # a copy of the rows, where the stream kernel makes none
            assert more >= (-(-F * dtype.itemsize // 128) * 128 * n_cols if not scaled else 1)
        _check_sums(Y[:, :F], row, col, n_active, X[:, :F], scale, dtype)
        untouched = torch.tensor(SENTINEL, dtype=dtype, device="cuda")
        assert (Y[n_active:] == untouched).all() and (Y[:, F:] == untouched).all()


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("form", ["two passes", "dist filter"])
def test_blocked_route_fours_of_several_slabs(form, dtype):
    """Scaled rows of several lines: sixteen blocks in two passes, or the entries that pass a filter.  Two passes also of the stream
    kernel, over a list of the same rows."""
    import paper_2311_06837_amd as P
    two, f32 = form == "two passes", dtype == torch.float32
    n_rows, n_cols = (38_000, 300_001) if two else (8_000, 70_001)
    longest = (460 if f32 else 580) if two else 1150
    F = 67 if two or f32 else 150
    G, row, col = _random_rows(n_rows, n_cols, longest, 7)
    gen = torch.Generator(device="cuda").manual_seed(8)
    ld = P.row_stride(F, dtype)
    X = torch.full((n_cols, ld), float("nan"), dtype=dtype, device="cuda")
    X[:, :F] = torch.randn(n_cols, F, generator=gen, device="cuda").to(dtype)
    scale = torch.rand(n_cols, generator=gen, device="cuda") + 0.5
    dist = None if two else (torch.arange(n_cols, device="cuda") % 3).int()
    Y = torch.full((n_rows, ld), SENTINEL, dtype=dtype, device="cuda")
    ws = P.Workspace()
    if two:
        P.gnn_masked_spmm_fwd(G, None, n_rows, X, Y, F, None, scale, ws=ws)
    else:
        P.gnn_masked_spmm_bwd(G, None, n_rows, dist, 1, X, Y, F, scale, None, accumulate=False, ws=ws)
        keep = dist[col] <= 1
        row, col = row[keep], col[keep]
    assert _used_blocked_route(ws) and ws.buf.numel() != _stream_bytes(G, n_rows, F, ld, dtype, True, not two, 16 if two else 8)
    _check_sums(Y[:, :F], row, col, n_rows, X[:, :F], scale, dtype)
    assert (Y[:, F:] == torch.tensor(SENTINEL, dtype=dtype, device="cuda")).all()
    if two:
        listed = torch.randperm(n_rows, generator=gen, device="cuda").int()
        Y.fill_(SENTINEL)
        ws = P.Workspace()
        P.gnn_masked_spmm_fwd(G, listed, n_rows, X, Y, F, ws=ws)
        assert ws.buf.numel() == _stream_bytes(G, n_rows, F, ld, dtype, False, False, 16)
        _check_sums(Y[:, :F], row, col, n_rows, X[:, :F], None, dtype)


def test_a_call_over_few_rows_needs_no_copy_of_the_matrix():
    """7500 rows of 400 entries over 150 000 ids, 256 floats: planes and ids, 90 MB, and no copy of the 154 MB of the gathered matrix."""
    import paper_2311_06837_amd as P
    n_rows, n_cols, F = 7500, 150_000, 256
    step = n_cols // 400
    col = torch.arange(400, device="cuda")[None] * step + torch.randint(step, (n_rows, 400), device="cuda")
    G = _graph(torch.arange(n_rows + 1, device="cuda") * 400, col.reshape(-1), n_cols)
    X, Y = torch.zeros(n_cols, F, device="cuda"), torch.zeros(n_rows, F, device="cuda")
    need = P.binding.spmm_workspace_bytes(G, n_rows, X, Y, F)
    assert 0 < need < X.numel() * 4


def test_blocked_route_falls_back_without_promise_or_density():
    """Unsorted columns (no GNN_CSR_SORTED_COLUMNS promise) or a sparse graph: the size query reports 0 and the
    call gathers whole rows."""
    import paper_2311_06837_amd as P
    g = _dense_graph()
    ws = P.Workspace()
    G = P.Graph(dev(g.row_ptr), dev(g.col_idx), sorted_columns=False)
    X = torch.randn(g.n_rows, 64, device="cuda")
    Y1, Y2 = torch.zeros_like(X), torch.zeros_like(X)
    P.gnn_masked_spmm_fwd(G, None, g.n_rows, X, Y1, 64, ws=ws)
    assert not _used_blocked_route(ws)
    Gs = P.Graph.from_numpy(g.row_ptr, g.col_idx)
    assert Gs.sorted_columns
    P.gnn_masked_spmm_fwd(Gs, None, g.n_rows, X, Y2, 64, ws=ws)
    assert _used_blocked_route(ws)
    assert (Y1 - Y2).abs().max() <= 1e-4 * Y1.abs().max()                 # the two routes differ by rounding order only
    sparse = gg.chung_lu(80000, 12.0, 2.1, 33)
    ws2 = P.Workspace()
    _fwd_case(sparse, 128, 128, torch.float32, None, True, 45, ws=ws2)
    assert not _used_blocked_route(ws2)


def test_blocked_route_backward_with_prefix_active_sources():
    """After a (distance, id) renumbering the forward rows are a PREFIX of the id range: every kept neighbour falls
    into the first stretch of ids.  The route balances its column blocks over the active vertices; results as ever."""
    import paper_2311_06837_amd as P
    g = _dense_graph()
    n, F = g.n_rows, 96
    rng = np.random.default_rng(77)
    n_fwd = 9000                                                          # forward rows 0 .. 8999
    dist = np.where(np.arange(n) < n_fwd, 0, 1).astype(np.int32)
    dY = as_stored(rng.standard_normal((n, F)), torch.float32)
    rs = (rng.random(n) + 0.5).astype(np.float32)
    cs = (rng.random(n) + 0.5).astype(np.float32)
    GT = P.Graph.from_numpy(g.row_ptr, g.col_idx)                         # symmetric
    ws = P.Workspace()
    dX = torch.full((n, F), SENTINEL, device="cuda")
    P.gnn_masked_spmm_bwd(GT, None, n, dev(dist), 0, dev(dY).float(), dX, F, dev(rs), dev(cs), accumulate=False, ws=ws)
    torch.cuda.synchronize()
    assert _used_blocked_route(ws)
    want = np.zeros((n, F))
    oracle.spmm_bwd(g.row_ptr, g.col_idx, np.arange(n_fwd, dtype=np.int32), dY, want, F, rs, cs)
    check(host64(dX), want, torch.float32, "prefix-active backward")


def _prefix_case(g, n_fwd, F, dtype, seed, sorted_promise=True, ws=None, accumulate=False, relu=False, out_rows=None):
    """Backward aggregation whose forward rows were the ids 0 .. n_fwd-1, told through src_prefix instead of a
    distance array.  The oracle gets the same thing as an explicit row list."""
    import paper_2311_06837_amd as P
    print(f"spmm bwd src_prefix: n={g.n_rows} nnz={g.nnz} n_fwd={n_fwd} F={F} {dtype} sorted={sorted_promise} acc={accumulate} "
          f"relu={relu}", flush=True)
    rng = np.random.default_rng(seed)
    n = g.n_rows
    gt = gg.transpose(g)
    dY = as_stored(rng.standard_normal((n, F)), dtype)
    rs = (rng.random(n) + 0.5).astype(np.float32)
    cs = (rng.random(n) + 0.5).astype(np.float32)
    init = as_stored(rng.standard_normal((n, F)), dtype) if accumulate else np.full((n, F), SENTINEL)
    Hact = as_stored(np.maximum(rng.standard_normal((n, F)), 0), dtype) if relu else None
    GT = P.Graph.from_numpy(gt.row_ptr, gt.col_idx)
    assert GT.sorted_columns
    if not sorted_promise:
        GT = P.Graph(GT.row_ptr, GT.col_idx, None, sorted_columns=False)     # same arrays, no promise: tested entry by entry
    rows_o = np.arange(n, dtype=np.int32) if out_rows is None else out_rows
    dXd = padded(init, F, dtype)
    P.gnn_masked_spmm_bwd(GT, None if out_rows is None else dev(rows_o), len(rows_o), None, 0, padded(dY, F, dtype), dXd, F, dev(rs),
                          dev(cs), accumulate=accumulate, ws=ws, relu_H=padded(Hact, F, dtype) if relu else None, src_prefix=n_fwd)
    torch.cuda.synchronize()
    want = np.zeros((n, F))
    oracle.spmm_bwd(g.row_ptr, g.col_idx, np.arange(n_fwd, dtype=np.int32), dY, want, F, rs, cs)
    if accumulate:
        want = want + init
    if relu:
        want = want * (Hact > 0)
    got = host64(dXd)
    check(got[rows_o], want[rows_o], dtype, "bwd rows")
    outside = np.setdiff1d(np.arange(n), rows_o)
    assert (got[outside] == host64(padded(init, F, dtype))[outside]).all(), "rows outside were written"


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("sorted_promise", [True, False])
def test_bwd_source_prefix(dtype, sorted_promise):
    g = gg.random_directed(8000, 6.0, 23)
    _prefix_case(g, 1500, 128, dtype, 31, sorted_promise)
    _prefix_case(g, 1, 64, dtype, 32, sorted_promise, accumulate=True)                 # a single forward row
    _prefix_case(g, 0, 64, dtype, 33, sorted_promise)                                  # none: every row sums to zero
    _prefix_case(g, 8000, 64, dtype, 34, sorted_promise, relu=True)                    # all: no cut at all
    _prefix_case(g, 7999, 100, dtype, 35, sorted_promise, accumulate=True, relu=True)
    rows = np.random.default_rng(36).permutation(8000)[:3001].astype(np.int32)
    _prefix_case(g, 4000, 7, dtype, 37, sorted_promise, out_rows=rows)
    h = gg.chung_lu(12000, 150.0, 2.1, 12)                                             # hub rows, cut inside the hub
    assert h.degrees().max() > 1200                                                    # (hub rows: longer than 1024)
    _prefix_case(h, 11000, 64, dtype, 38, sorted_promise, relu=True)                   # still hubs after the cut
    _prefix_case(h, 11000, 16, dtype, 40, sorted_promise)
    _prefix_case(h, 6000, 64, dtype, 39, sorted_promise)                               # hubs that stop being hubs after the cut


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_blocked_route_backward_with_source_prefix(dtype):
    """The column-blocked route cuts its blocks out of [0, src_prefix) only."""
    import paper_2311_06837_amd as P
    g = _dense_enough(dtype)
    ws = P.Workspace()
    _prefix_case(g, 68001, 96, dtype, 78, ws=ws, relu=True)          # 68001 * 256 B is still above the route's threshold
    assert _used_blocked_route(ws)
    _prefix_case(g, 66000, 200, dtype, 79, ws=ws, accumulate=True)
    ws2 = P.Workspace()
    _prefix_case(g, 9000, 96, dtype, 80, ws=ws2)                     # a short prefix fits the caches: one launch
    assert not _used_blocked_route(ws2)


@pytest.mark.parametrize("form", ["all rows", "row list", "source prefix", "distances"])
def test_blocked_route_gives_the_dies_equal_shares(form):
    """Every column block holds about the same number of the call's entries, wherever in the id range they lie: the die whose
    block has most ends last.  Here the first eighth of the ids draws a third of the entries (equal ids: 3.1 shares).  The cut
    points of the rows are the first array of the workspace."""
    import paper_2311_06837_amd as P
    n, F = 70_000, 64
    rng = np.random.default_rng(19)
    row = np.repeat(np.arange(n, dtype=np.int64), 120)
    col = np.where(rng.random(len(row)) < 0.3, rng.integers(0, n // 8, len(row)), rng.integers(0, n, len(row)))
    keys = np.unique(row * n + col)
    row, col = keys // n, (keys % n).astype(np.int32)
    row_ptr = np.zeros(n + 1, np.int32)
    row_ptr[1:] = np.cumsum(np.bincount(row, minlength=n))
    G = P.Graph.from_numpy(row_ptr, col)
    X = torch.randn(n, F, device="cuda")
    Y, Z = torch.zeros_like(X), torch.zeros_like(X)
    ws = P.Workspace()
    rows, dist, prefix = None, None, -1
    kept = np.ones(len(col), bool)
    if form == "row list":
        rows = rng.permutation(n)[: n // 2].astype(np.int32)
    elif form == "source prefix":
        prefix = 68_001
        kept = col < prefix
    elif form == "distances":
        dist = rng.integers(0, 3, n).astype(np.int32)
        kept = dist[col] <= 1
    n_out = n if rows is None else len(rows)

    def call(out, w):
        P.gnn_masked_spmm_bwd(G, dev(rows) if rows is not None else None, n_out, dev(dist) if dist is not None else None, 1, X, out, F, None, None,
                              accumulate=False, ws=w, src_prefix=prefix)
    call(Y, ws)
    call(Z, None)
    assert _used_blocked_route(ws)
    seg = ws.buf[: n_out * 9 * 4].view(torch.int32).reshape(n_out, 9).cpu().numpy()
    before = np.concatenate([[0], np.cumsum(kept)])
    share = (before[seg[:, 1:]] - before[seg[:, :-1]]).sum(0)
    print(form, (share / share.mean()).round(3), flush=True)
    # a block's share of 65 536 samples: 1 % of itself at one standard deviation, 1.3 % where two thirds of them pass the filter
    assert share.max() <= 1.06 * share.mean() and share.min() >= 0.94 * share.mean()
    assert (Y - Z).abs().max() <= 1e-4 * Z.abs().max()


def test_die_mapping_probe_and_the_route_that_depends_on_it():
    """Workgroup i on compute die i mod 8: the probe's raw ids are checked here on the CPU, and the size query of a call the
    column-blocked route is made for offers the route exactly when the pattern holds."""
    import paper_2311_06837_amd as P
    ids, holds = P.gnn_die_mapping()
    print("die ids of the probe grid:", ids, flush=True)
    assert len(ids) == 64 and all(0 <= i < 8 for i in ids)
    pattern = len(set(ids[:8])) == 8 and all(ids[i] == ids[i % 8] for i in range(64))
    assert holds == pattern
    g = gg.chung_lu(80_000, 160.0, 2.1, 17)       # dense enough: 20 entries of a row per column block, an 20 MB slab
    G = P.Graph.from_numpy(g.row_ptr, g.col_idx)
    X = torch.zeros(g.n_rows, 64, device="cuda")
    need = P.binding.spmm_workspace_bytes(G, g.n_rows, X, X.clone(), 64)
    assert (need > 0) == pattern
