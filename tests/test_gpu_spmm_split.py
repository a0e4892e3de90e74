"""The split route of the aggregation (hot neighbours summed from a table, the others by the row kernel), against plain torch
sums in 64 bits, at the places where its pieces meet: chunks of 8192 entries, fours of slots, rows that cross chunks, runs of
rows without entries, a cut at a source prefix, slabs of 32 columns."""
import numpy as np
import pytest
import torch

import graphgen as gg

pytestmark = pytest.mark.gpu
CTRL = 256 * 256 * 4 + 256 * 4      # byte offset in the workspace of (hot neighbours, 1: the route went on)


def _graph(n, deg, seed, empty=(), hubs=0):
    """Skewed, symmetric but for the rows of `empty` (ranges), whose entries are dropped, and the first `hubs` rows, which hold
    30 000 entries more."""
    g = gg.chung_lu(n, deg, 2.1, seed)
    rng = np.random.default_rng(seed)
    rows = np.repeat(np.arange(n, dtype=np.int64), g.degrees())
    keys = rows * n + g.col_idx
    keep = np.ones(len(keys), bool)
    for a, b in empty:
        keep &= (rows < a) | (rows >= b)
    keys = keys[keep]
    for r in range(hubs):
        keys = np.concatenate([keys, r * n + rng.integers(0, n, 30_000)])
    keys = np.unique(keys)
    row_ptr = np.zeros(n + 1, np.int64)
    row_ptr[1:] = np.cumsum(np.bincount(keys // n, minlength=n))
    return row_ptr.astype(np.int32), (keys % n).astype(np.int32)


def _want(row_ptr, ci, n_active, X, rs, cs, limit):
    """-> the sums in 64 bits, and the sums of the magnitudes."""
    F = X.shape[1]
    out, size = (torch.zeros(n_active, F, dtype=torch.float64, device="cuda") for _ in range(2))
    m = int(row_ptr[n_active])
    lens = torch.from_numpy(np.diff(row_ptr[: n_active + 1]).astype(np.int64)).cuda()
    row = torch.repeat_interleave(torch.arange(n_active, device="cuda"), lens)
    for a in range(int(row_ptr[0]), m, 400_000):
        b = min(m, a + 400_000)
        r, c = row[a - int(row_ptr[0]): b - int(row_ptr[0])], ci[a:b].long()
        ok = c < limit
        r, c = r[ok], c[ok]
        t = X[c].double() * (cs[c].double()[:, None] if cs is not None else 1.0)
        out.index_add_(0, r, t)
        size.index_add_(0, r, t.abs())
    s = rs[:n_active].double()[:, None] if rs is not None else 1.0
    return out * s, size * s, lens[:, None].double()


CASES = {
    # name: graph arguments, F, ld, scales, rows (share), source prefix (share), accumulate and ReLU
    "256": (dict(n=60_000, deg=46, seed=1), 256, 256, True, 1.0, None, False),
    "100_crossing_rows": (dict(n=140_001, deg=60, seed=2, hubs=3, empty=((40, 7000), (100_000, 101_500))), 100, 128, False, 0.83, None, False),
    "301_prefix": (dict(n=50_000, deg=50, seed=3, hubs=2, empty=((30_000, 34_000),)), 301, 304, True, 1.0, 0.9, True),
    "97_prefix": (dict(n=400_000, deg=45, seed=4, empty=((0, 2500),)), 97, 100, True, 0.999, 0.97, False),
    "640": (dict(n=24_000, deg=50, seed=5, hubs=1), 640, 640, True, 1.0, None, True),
    "800_two_column_blocks": (dict(n=24_000, deg=50, seed=6, hubs=1), 800, 800, True, 1.0, None, False),
    "few_rows": (dict(n=140_000, deg=60, seed=7, hubs=1), 256, 256, True, 0.06, None, True),
    "short_prefix": (dict(n=140_000, deg=60, seed=8, hubs=1), 256, 256, True, 1.0, 0.37, False),
}


@pytest.mark.parametrize("name", list(CASES))
def test_split_route(name):
    import paper_2311_06837_amd as P
    kw, F, ld, scales, share, prefix, extra = CASES[name]
    dtype = torch.float32
    row_ptr, col = _graph(**kw)
    n, n_active = kw["n"], int(kw["n"] * share)
    G = P.Graph(torch.from_numpy(row_ptr).cuda(), torch.from_numpy(col).cuda(), sorted_columns=True)
    gen = torch.Generator(device="cuda").manual_seed(7)
    X = torch.full((n, ld), float("nan"), dtype=dtype, device="cuda")                 # pad columns must never matter
    X[:, :F] = torch.randn(n, F, generator=gen, device="cuda").to(dtype)
    limit = n if prefix is None else int(n * prefix)
    rs, cs = ((torch.rand(n, generator=gen, device="cuda") + 0.5) if scales else None for _ in range(2))
    Y = torch.full((n, ld), 12345.0, dtype=dtype, device="cuda")
    H = None
    if extra:
        Y[:, :F] = torch.randn(n, F, generator=gen, device="cuda").to(dtype)
        H = torch.randn(n, ld, generator=gen, device="cuda").to(dtype)
    start = Y.clone()
    ws = P.Workspace()

    def call(w):
        Y.copy_(start)
        if prefix is None and not extra:
            P.gnn_masked_spmm_fwd(G, None, n_active, X, Y, F, rs, cs, ws=w)
        else:
            P.gnn_masked_spmm_bwd(G, None, n_active, None, 0, X, Y, F, cs, rs, accumulate=extra, ws=w, relu_H=H, src_prefix=-1 if prefix is None else limit)
        return Y.clone()

    got = call(ws)
    n_hot, on = ws.buf[CTRL: CTRL + 8].view(torch.int32).tolist()
    print(f"{name}: {len(col)} entries, {n_hot} hot neighbours", flush=True)
    assert on == 1 and 0 < n_hot <= 65535
    want, size, lens = _want(row_ptr, torch.from_numpy(col).cuda(), n_active, X[:, :F], rs, cs, limit)
    if extra:
        want = torch.where(H[:n_active, :F] > 0, want + start[:n_active, :F].double(), 0.0)
        size = size + start[:n_active, :F].double().abs()
    # fp32 sums in any order with two roundings more a term: at most (terms + 8) * 2^-24 of the sum of magnitudes
    tol = (lens + 8) * 2.0 ** -24 * size + 1e-30
    worst = ((got[:n_active, :F].double() - want).abs() / tol).max().item()
    assert worst <= 1.0, worst
    assert torch.equal(got[n_active:], start[n_active:]) and torch.equal(got[:, F:], start[:, F:]), "written outside"
    assert torch.equal(call(ws), got), "not the same bits twice"
    small = P.Workspace()
    small.buf = torch.empty(4096, dtype=torch.uint8, device="cuda")
    plain = call(None)
    lib, C = P.binding.lib(), P.binding.C          # a workspace too small for the route: as without one
    Y.copy_(start)
    P.binding._check(lib.gnn_masked_spmm_bwd(C.byref(G.c), None, n_active, None, 0, -1 if prefix is None else limit, X.data_ptr(), ld, Y.data_ptr(), ld, F,
                                             0, cs.data_ptr() if scales else None, rs.data_ptr() if scales else None,
                                             1 if extra else 0, H.data_ptr() if extra else None, ld if extra else 0,
                                             small.buf.data_ptr(), C.byref(C.c_size_t(4096)), P.binding._stream()))
    assert torch.equal(Y, plain)


def _sum_and_bound(row_ptr, col, n, X, rs, cs, extra):
    """64-bit sums plus `extra`, and what fp32 sums in any order may be off by."""
    want, size, lens = _want(row_ptr, torch.from_numpy(col).cuda(), n, X, rs, cs, X.shape[0])
    return want + extra.double(), (lens + 8) * 2.0 ** -24 * (size + extra.double().abs()) + 1e-30


@pytest.mark.parametrize("bias", [False, True])
@pytest.mark.parametrize("relu", [False, True])
def test_split_route_added_onto_the_output(bias, relu):
    """gnn_masked_spmm_fwd_add: the rows start from what Y holds or from a bias, the ReLU's matrix is Y itself."""
    import paper_2311_06837_amd as P
    n, F = 60_000, 252
    row_ptr, col = _graph(n, 46, 1, hubs=2, empty=((30_000, 31_000),))
    G = P.Graph(torch.from_numpy(row_ptr).cuda(), torch.from_numpy(col).cuda(), sorted_columns=True)
    gen = torch.Generator(device="cuda").manual_seed(3)
    X, Y = (torch.randn(n, F, generator=gen, device="cuda") for _ in range(2))
    rs, cs = (torch.rand(n, generator=gen, device="cuda") + 0.5 for _ in range(2))
    b = torch.randn(F, generator=gen, device="cuda") if bias else None
    want, tol = _sum_and_bound(row_ptr, col, n, X, rs, cs, b[None].expand(n, F) if bias else Y)
    ws = P.Workspace()
    P.gnn_masked_spmm_fwd_add(G, None, n, X, Y, F, rs, cs, relu=relu, ws=ws, bias=b)
    assert ws.buf[CTRL: CTRL + 8].view(torch.int32).tolist()[1] == 1
    want = torch.relu(want) if relu else want
    assert ((Y.double() - want).abs() / tol).max().item() <= 1.0


def test_split_route_with_infinities_and_nan():
    """In frequent neighbours (the table) and in others: a sum is infinite or NaN where it is without the route, the rest are untouched."""
    import paper_2311_06837_amd as P
    n, F = 60_000, 256
    row_ptr, col = _graph(n, 46, 1)
    G = P.Graph(torch.from_numpy(row_ptr).cuda(), torch.from_numpy(col).cuda(), sorted_columns=True)
    lens = np.diff(row_ptr)
    often, seldom = np.argsort(-lens)[:3], np.flatnonzero(lens == lens[lens > 0].min())[:3]
    X = torch.randn(n, F, device="cuda")
    for a, b, c in (often, seldom):
        X[a, 5], X[b, 7], X[b, 9], X[c, 9] = float("inf"), float("nan"), float("inf"), float("-inf")
    Y, Z = torch.zeros_like(X), torch.zeros_like(X)
    ws = P.Workspace()
    P.gnn_masked_spmm_fwd(G, None, n, X, Y, F, ws=ws)
    P.gnn_masked_spmm_fwd(G, None, n, X, Z, F)
    assert ws.buf[CTRL: CTRL + 8].view(torch.int32).tolist()[1] == 1
    assert torch.equal(torch.isnan(Y), torch.isnan(Z)) and torch.equal(torch.isinf(Y), torch.isinf(Z))
    assert torch.isnan(Y).any() and torch.isinf(Y).any()
    ok = torch.isfinite(Z)
    assert torch.equal(torch.sign(Y[torch.isinf(Y)]), torch.sign(Z[torch.isinf(Z)])) and (Y[ok] - Z[ok]).abs().max() <= 1e-4 * Z[ok].abs().max()


def test_split_route_over_the_last_rows_of_a_graph():
    """A row pointer that does not begin at 0: the rows behind the first of a larger graph."""
    import paper_2311_06837_amd as P
    n, F, first = 120_000, 128, 3001
    row_ptr, col = _graph(n, 60, 9)
    assert row_ptr[first] > 8192
    G = P.Graph(torch.from_numpy(row_ptr[first:]).cuda(), torch.from_numpy(col).cuda(), n_cols=n, sorted_columns=True)
    X = torch.randn(n, F, device="cuda")
    Y = torch.zeros(n - first, F, device="cuda")
    ws = P.Workspace()
    P.gnn_masked_spmm_fwd(G, None, n - first, X, Y, F, ws=ws)
    on = ws.buf[CTRL: CTRL + 8].view(torch.int32).tolist()[1]
    want, tol = _sum_and_bound(row_ptr[first:], col, n - first, X, None, None, torch.zeros_like(Y))
    print("went on:", on, flush=True)
    assert ((Y.double() - want).abs() / tol).max().item() <= 1.0


@pytest.mark.parametrize("skewed_rows", [False, True])
def test_a_graph_without_hot_neighbours_runs_as_before(skewed_rows):
    """Every neighbour equally frequent: seen from the row lengths, or, where those are skewed, from the samples."""
    import paper_2311_06837_amd as P
    n, deg, F = 400_000, 42, 128
    rng = np.random.default_rng(3)
    lens = np.minimum(rng.pareto(1.1, n) * 12 + 1, 20_000).astype(np.int64) if skewed_rows else np.full(n, deg)
    lens = np.maximum(1, lens * deg * n // lens.sum())
    rows = np.repeat(np.arange(n, dtype=np.int64), lens)
    keys = np.unique(rows * n + rng.integers(0, n, len(rows)))
    row_ptr = np.zeros(n + 1, np.int64)
    row_ptr[1:] = np.cumsum(np.bincount(keys // n, minlength=n))
    assert len(keys) // n >= 40
    G = P.Graph(torch.from_numpy(row_ptr.astype(np.int32)).cuda(), torch.from_numpy((keys % n).astype(np.int32)).cuda(), sorted_columns=True)
    X = torch.randn(n, F, device="cuda")
    ws = P.Workspace()
    Y, Z = torch.zeros_like(X), torch.zeros_like(X)
    P.gnn_masked_spmm_fwd(G, None, n, X, Y, F, ws=ws)
    P.gnn_masked_spmm_fwd(G, None, n, X, Z, F)
    n_hot, on = ws.buf[CTRL: CTRL + 8].view(torch.int32).tolist()
    assert on == 0 and (n_hot > 0) == skewed_rows
    assert torch.equal(Y, Z)


def test_dies_share_the_chunks_in_use():
    """A call over the first half of the rows: the table's sums are dealt to the dies by the chunks that these rows' entries fill
    (dealt by all chunks of the graph, half of the dies had nothing to do: 554 us with the route, 453 without; now 441)."""
    import paper_2311_06837_amd as P
    n, F = 300_000, 128
    row_ptr, col = _graph(n, 50, 6)
    G = P.Graph(torch.from_numpy(row_ptr).cuda(), torch.from_numpy(col).cuda(), sorted_columns=True)
    X = torch.randn(n, F, device="cuda")
    Y, ws = torch.zeros_like(X), P.Workspace()

    def time_us(w):
        times = []
        for _ in range(6):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(5):
                P.gnn_masked_spmm_fwd(G, None, n // 2, X, Y, F, ws=w)
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b) * 200)
        return min(times)
    split, plain = time_us(ws), time_us(None)
    assert ws.buf[CTRL: CTRL + 8].view(torch.int32).tolist()[1] == 1
    print(f"split route {split:.0f} us, row kernel {plain:.0f} us", flush=True)
    assert split < 1.08 * plain      # between the two


@pytest.mark.parametrize("n,deg,F,rows,prefix,takes", [
    (1_200_000, 51, 256, 1.0, 1.0, True), (1_200_000, 51, 256, 0.05, 1.0, True), (1_200_000, 51, 256, 0.004, 1.0, False),
    (1_200_000, 51, 100, 0.05, 1.0, True), (1_200_000, 51, 100, 0.01, 1.0, False), (300_000, 51, 128, 0.05, 1.0, False),
    (1_200_000, 51, 256, 1.0, 0.5, True), (1_200_000, 51, 256, 1.0, 0.125, True), (1_200_000, 51, 256, 1.0, 0.1, False), (1_200_000, 51, 100, 1.0, 0.25, False),
    (300_000, 51, 256, 0.1, 0.5, False), (300_000, 51, 256, 1.0, 0.5, True), (1_200_000, 39, 256, 1.0, 1.0, False)])
def test_the_route_is_asked_for_by_the_work_of_the_call(n, deg, F, rows, prefix, takes):
    """Few rows, or a source prefix that leaves little of them, are not worth the route's look at all neighbours.  A size query reads
    no array, so none is made."""
    import paper_2311_06837_amd as P
    C, some = P.binding.C, torch.zeros(64, device="cuda")
    g = P.binding.gnn_csr(n, n, n * deg, some.data_ptr(), some.data_ptr(), P.binding.GNN_CSR_SORTED_COLUMNS, None)
    need = C.c_size_t(0)
    P.binding._check(P.binding.lib().gnn_masked_spmm_bwd(
        C.byref(g), None, int(n * rows), None, 0, -1 if prefix == 1.0 else int(n * prefix), some.data_ptr(), F, some.data_ptr(), F, F, 0, None, None, 0,
        None, 0, None, C.byref(need), P.binding._stream()))
    assert (need.value > 0) == takes


def _full_card(monkeypatch, limit):
    """An allocator that has nothing of more than `limit` bytes; -> the sizes it was asked for."""
    import paper_2311_06837_amd.binding as B
    asked, empty = [], torch.empty

    def few(*size, **kw):
        if kw.get("dtype") == torch.uint8:
            asked.append(size[0])
            if size[0] > limit:
                raise torch.cuda.OutOfMemoryError("none left")
        return empty(*size, **kw)
    monkeypatch.setattr(B.torch, "empty", few)
    return asked


@pytest.mark.parametrize("why", ["no room", "in pieces", "capture"])
def test_without_memory_for_the_route(why, monkeypatch):
    """The route's workspace is one the call can do without: it is not taken from a card where half of what is left would not hold it,
    not while a stream captures, and a card that has none is not asked at every call."""
    import paper_2311_06837_amd as P
    import paper_2311_06837_amd.binding as B
    n, F = 60_000, 256
    row_ptr, col = _graph(n, 46, 1)
    G = P.Graph(torch.from_numpy(row_ptr).cuda(), torch.from_numpy(col).cuda(), sorted_columns=True)
    X = torch.randn(n, F, device="cuda")
    Y, Z = torch.zeros_like(X), torch.zeros_like(X)
    need = B.spmm_workspace_bytes(G, n, X, Y, F)
    assert need > 1 << 20
    P.gnn_masked_spmm_fwd(G, None, n, X, Z, F)
    ws = P.Workspace()
    call = lambda: P.gnn_masked_spmm_fwd(G, None, n, X, Y, F, ws=ws)
    if why == "capture":
        graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
        with torch.cuda.graph(graph, stream=side):
            call()
        assert ws.buf.numel() == 256
        for _ in range(3):
            Y.zero_()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(Y, Z)
        return
    asked = _full_card(monkeypatch, 1 << 20 if why == "in pieces" else 1 << 40)
    if why == "no room":
        left = 2 * need - 1
        monkeypatch.setattr(torch.cuda, "mem_get_info", lambda: (left // 2, 1 << 40))
        monkeypatch.setattr(torch.cuda, "memory_reserved", lambda: left - left // 2 + (1 << 20))
        monkeypatch.setattr(torch.cuda, "memory_allocated", lambda: 1 << 20)
    for _ in range(100):
        call()
    assert asked == ([256] if why == "no room" else [need, 256])
    assert torch.equal(Y, Z)
    monkeypatch.undo()
    for _ in range(200):        # memory is there again
        call()
    assert ws.buf.numel() >= need


def test_a_route_that_insists_on_its_workspace_still_does(monkeypatch):
    """The column-blocked route raises where there is no memory for it."""
    import paper_2311_06837_amd as P
    n, F = 70_000, 256
    rng = np.random.default_rng(2)
    keys = np.unique(np.repeat(np.arange(n, dtype=np.int64), 80) * n + rng.integers(0, n, 80 * n))
    row_ptr = np.zeros(n + 1, np.int32)
    row_ptr[1:] = np.cumsum(np.bincount(keys // n, minlength=n))
    G = P.Graph.from_numpy(row_ptr, (keys % n).astype(np.int32))
    X = torch.randn(n, F, device="cuda")
    assert P.binding.spmm_workspace_bytes(G, n, X, X.clone(), F) >= 8 * n * F * 4
    ws, Y = P.Workspace(), torch.zeros_like(X)
    _full_card(monkeypatch, 1 << 20)
    with pytest.raises(torch.cuda.OutOfMemoryError):
        P.gnn_masked_spmm_fwd(G, None, n, X, Y, F, ws=ws)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_without_memory_for_the_copy_of_the_rows(dtype, monkeypatch):
    """A workspace that does not hold the copy of the gathered rows and the streams of fours, but what the stream kernel needs: the call takes
    that, as it does for a list of the same rows, and one byte less is an error; on a card with so much the binding finds it."""
    import paper_2311_06837_amd as P
    n, F = 66_000, 256
    rng = np.random.default_rng(2)
    keys = np.unique(np.repeat(np.arange(n, dtype=np.int64), 140) * n + rng.integers(0, n, 140 * n))
    row_ptr = np.zeros(n + 1, np.int32)
    row_ptr[1:] = np.cumsum(np.bincount(keys // n, minlength=n))
    G = P.Graph.from_numpy(row_ptr, (keys % n).astype(np.int32))
    X = torch.randn(n, F, device="cuda").to(dtype)
    Y, Z = torch.zeros_like(X), torch.zeros_like(X)
    list_ws = P.Workspace()
    P.gnn_masked_spmm_fwd(G, torch.arange(n, device="cuda").int(), n, X, Z, F, ws=list_ws)
    small, need = list_ws.buf.numel(), P.binding.spmm_workspace_bytes(G, n, X, Y, F)
    assert 256 < small < need - X.numel() * X.element_size()
    lib, C = P.binding.lib(), P.binding.C
    for size, status in ((small - 256, P.binding.GNN_ERR_WORKSPACE), (small, 0)):
        got = lib.gnn_masked_spmm_fwd(C.byref(G.c), None, n, X.data_ptr(), F, Y.data_ptr(), F, F, P.binding._dtype_code(X), None, None,
                                      list_ws.buf.data_ptr(), C.byref(C.c_size_t(size)), P.binding._stream())
        assert got == status
    assert torch.equal(Y, Z)
    Y.zero_()
    ws = P.Workspace()
    asked = _full_card(monkeypatch, need - 1)
    monkeypatch.setattr(torch.cuda, "mem_get_info", lambda: (need, 1 << 40))
    for _ in range(3):
        P.gnn_masked_spmm_fwd(G, None, n, X, Y, F, ws=ws)
    assert torch.equal(Y, Z) and small <= ws.buf.numel() < need
    print(asked, small, need, flush=True)
    monkeypatch.undo()
    for _ in range(300):        # memory is there again
        P.gnn_masked_spmm_fwd(G, None, n, X, Y, F, ws=ws)
    assert ws.buf.numel() == need
    assert (Y.float() - Z.float()).abs().max() <= (1e-4 if dtype == torch.float32 else 2e-2) * Z.float().abs().max()


def test_a_workspace_gives_its_buffer_back_before_it_grows():
    import paper_2311_06837_amd as P
    ws = P.Workspace()
    ws.get(64 << 20)
    torch.cuda.empty_cache()
    torch.cuda.reset_peak_memory_stats()
    before = torch.cuda.memory_allocated()
    ws.get(96 << 20)
    assert torch.cuda.max_memory_allocated() <= before + (40 << 20)


@pytest.mark.parametrize("graph,dtype,route", [("skewed", torch.float32, "split"), ("even", torch.float32, "rows"), ("skewed", torch.bfloat16, "rows"),
                                               ("dense", torch.float32, "columns"), ("dense", torch.bfloat16, "columns")])
def test_the_route_that_a_call_took(graph, dtype, route):
    """Asked before the call, the route it prepares for; with the call's workspace, the one it went on with."""
    import paper_2311_06837_amd as P
    if graph == "skewed":
        n, (row_ptr, col) = 60_000, _graph(60_000, 46, 1)
    else:
        n, deg = (140_000, 46) if graph == "even" else (70_000, 80 if dtype == torch.float32 else 120)
        rng = np.random.default_rng(2)
        keys = np.unique(np.repeat(np.arange(n, dtype=np.int64), deg) * n + rng.integers(0, n, deg * n))
        row_ptr, col = np.searchsorted(keys, np.arange(n + 1, dtype=np.int64) * n).astype(np.int32), (keys % n).astype(np.int32)
    G = P.Graph(torch.from_numpy(row_ptr).cuda(), torch.from_numpy(col).cuda(), sorted_columns=True)
    X = torch.randn(n, 256, device="cuda").to(dtype)
    Y, ws = torch.zeros_like(X), P.Workspace()
    before = P.gnn_spmm_route(G, None, n, X, Y, 256)
    assert before == ("split" if graph != "dense" and dtype == torch.float32 else route)
    P.gnn_masked_spmm_fwd(G, None, n, X, Y, 256, ws=ws)
    assert P.gnn_spmm_route(G, None, n, X, Y, 256, ws=ws) == route
    assert P.gnn_spmm_route(G, None, 100, X, Y, 256) == "rows"
