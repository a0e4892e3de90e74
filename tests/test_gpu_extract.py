"""GPU parity: gnn_extract_partition and gnn_gather_rows against the oracle (section 6 step 1: the one-hop graph
of the traversed vertices, renumbered by (distance, id)).  Integer outputs are compared bit-exact."""
import numpy as np
import pytest
import torch

import graphgen as gg
import oracle
from gpu_util import TOL, backward_at_the_oracles_point, check, dev

pytestmark = pytest.mark.gpu


def _extract_case(g, T, L, what):
    import paper_2311_06837_amd as P
    print(f"extract: {what} n={g.n_rows} nnz={g.nnz} |T|={len(T)} L={L}", flush=True)
    G = P.Graph.from_numpy(g.row_ptr, g.col_idx)
    ws = P.Workspace()
    dist, ring, hop_d, hop = P.gnn_build_active_sets(G, dev(np.asarray(T, dtype=np.int32)), L, ws=ws)
    n_local = int(hop[-1])
    local, new_id = P.gnn_extract_partition(G, ring, n_local, dist, L, ws=ws)
    torch.cuda.synchronize()
    rp, ci, l2g, off, dl = oracle.extract_partition(g.row_ptr, g.col_idx, T, L)
    assert n_local == l2g.size and list(hop) == list(off)
    assert np.array_equal(ring.cpu().numpy()[:n_local], l2g)
    assert np.array_equal(local.row_ptr.cpu().numpy(), rp)
    assert np.array_equal(local.col_idx.cpu().numpy(), ci)
    want_new = np.full(g.n_rows, -1, dtype=np.int32)
    want_new[l2g] = np.arange(l2g.size, dtype=np.int32)
    assert np.array_equal(new_id.cpu().numpy(), want_new)
    assert local.sorted_columns and local.n_rows == n_local and local.nnz == ci.size
    return local, ring, hop, (rp, ci, l2g, off, dl)


@pytest.mark.parametrize("L", [1, 2, 3])
def test_power_law_graph_with_hubs(L):
    g = gg.chung_lu(30000, 40.0, 2.1, 51)                     # hub rows of > 1000 entries
    T = np.sort(np.random.default_rng(L).choice(30000, 300, replace=False))
    _extract_case(g, T, L, "chung-lu")


def test_directed_graph_deep_and_unreached_vertices():
    g = gg.random_directed(20000, 1.5, 52)                    # many empty rows, most vertices never reached
    T = np.sort(np.random.default_rng(2).choice(20000, 50, replace=False))
    local, ring, hop, (rp, ci, l2g, off, dl) = _extract_case(g, T, 8, "directed")
    assert l2g.size < 20000


def test_whole_graph_is_traversed_and_degenerate_sizes():
    import paper_2311_06837_amd as P
    g = gg.erdos_renyi(5000, 12.0, 53)
    _extract_case(g, np.arange(0, 5000, 7), 4, "everything reached")
    _extract_case(g, np.array([17]), 1, "one target")
    # n_local = 0: an empty graph comes back
    G = P.Graph.from_numpy(g.row_ptr, g.col_idx)
    dist = torch.full((5000,), -1, dtype=torch.int32, device="cuda")
    ring = torch.zeros(1, dtype=torch.int32, device="cuda")
    local, new_id = P.gnn_extract_partition(G, ring, 0, dist, 2)
    assert local.n_rows == 0 and local.nnz == 0 and int(local.row_ptr[0]) == 0 and bool((new_id == -1).all())


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("F,ld_src,ld_dst", [(64, 64, 64), (602, 608, 608), (100, 100, 128), (7, 7, 9)])
def test_gather_rows(dtype, F, ld_src, ld_dst):
    import paper_2311_06837_amd as P
    rng = np.random.default_rng(F)
    n_src, n = 4000, 2501
    src = torch.randn(n_src, ld_src, device="cuda").to(dtype)
    ids = rng.integers(0, n_src, size=n).astype(np.int32)
    dst = torch.full((n, ld_dst), 7.0, dtype=dtype, device="cuda")
    P.gnn_gather_rows(src, dev(ids), F, dst)
    torch.cuda.synchronize()
    assert torch.equal(dst[:, :F], src[torch.from_numpy(ids).cuda().long(), :F])
    if ld_dst > F:
        assert bool((dst[:, F:] == 7.0).all()), "pad columns were written"


@pytest.mark.parametrize("kind,dtype", [("sage", torch.float32), ("gcn", torch.float32), ("sage", torch.bfloat16)])
def test_training_step_on_the_extracted_graph(kind, dtype):
    """The whole chain on the GPU - active sets of the unpartitioned graph, extraction, feature gather, one training
    step with prefix row sets - against the oracle's model on the oracle's extraction."""
    import paper_2311_06837_amd as P
    n, L, dims = 20000, 3, [48, 32, 32, 7]
    g = gg.chung_lu(n, 14.0, 2.1, 61)
    if kind == "gcn":
        g = gg.add_self_loops(g)
    rng = np.random.default_rng(61)
    T = np.sort(rng.choice(n, 150, replace=False))
    local, ring, hop, (rp, ci, l2g, off, dl) = _extract_case(g, T, L, f"model {kind}")
    n_local = l2g.size
    assert n_local < n
    params = gg.layer_weights(dims, kind == "sage", 61)
    H0g = gg.features(n, dims[0], 61)
    y = gg.labels(len(T), dims[-1], 61)

    bf16 = dtype == torch.bfloat16
    H0o = oracle.round_bf16(H0g.astype(np.float64)) if bf16 else H0g.astype(np.float64)
    om = oracle.Model(rp, ci, np.arange(len(T), dtype=np.int32), kind, params, g.degrees()[l2g] if kind == "gcn" else None, bf16=bf16)
    loss_o = om.forward(H0o[l2g], y)
    grads_o = om.backward()

    ld0 = P.row_stride(dims[0], dtype)
    H0d = torch.zeros(n_local, ld0, dtype=dtype, device="cuda")
    P.gnn_gather_rows(dev(H0g).to(dtype), ring[:n_local], dims[0], H0d)
    m = P.MaskedGNN(local, local, torch.arange(len(T), dtype=torch.int32, device="cuda"), kind,
                    [{k: dev(v) for k, v in p.items()} for p in params], dtype=dtype,
                    global_degree=dev(g.degrees()[l2g].astype(np.int32)) if kind == "gcn" else None,
                    prefix_numbered=True,     # the extraction numbers by (distance, id): the calls get rows = NULL
                    transform_first=kind == "sage")   # and the narrowing GraphSAGE layers run in the exchanged order
    m.set_input(H0d)
    loss = m.step(dev(y))
    torch.cuda.synchronize()
    assert list(m.hop) == list(off)
    assert torch.equal(m.ring_ids[:n_local].cpu(), torch.arange(n_local, dtype=torch.int32))   # the numbering IS the ring order
    tol = TOL[dtype] * 2 * L
    assert abs(loss.item() - loss_o) <= tol * abs(loss_o), (loss.item(), loss_o)
    backward_at_the_oracles_point(m, om, dims, dtype, dev(y))     # same ReLU decisions on both sides, then element by element
    for l, gr in enumerate(grads_o):
        for k, want in gr.items():
            check(m.grads[l][k].double().cpu().numpy(), want, dtype, f"layer {l + 1} {k}", calls=L - l)


# ---- extraction after boundary sampling ----------------------------------------------------------------------

def _sampled_case(g, T, fanout, seed, what):
    import paper_2311_06837_amd as P
    print(f"extract sampled: {what} n={g.n_rows} nnz={g.nnz} |T|={len(T)} fanout={fanout}", flush=True)
    n = g.n_rows
    G = P.Graph.from_numpy(g.row_ptr, g.col_idx)
    Td = dev(np.asarray(T, dtype=np.int32))
    bits = P.gnn_make_bitmap(Td, n)
    ws = P.Workspace()
    srp, sci = P.gnn_sample_boundary(G, bits, Td, fanout, seed, ws=ws)
    local, l2g_d, hop = P.gnn_extract_sampled_partition(G, Td, srp, sci, ws=ws)      # symmetric graph: gT = g
    torch.cuda.synchronize()
    is_t = np.zeros(n, dtype=np.uint8)
    is_t[T] = 1
    osrp, osci = oracle.sample_boundary(g.row_ptr, g.col_idx, is_t, T, fanout, seed)
    rp, ci, l2g, off, dl = oracle.extract_sampled(n, T, osrp, osci)
    assert list(hop) == list(off)
    assert np.array_equal(l2g_d.cpu().numpy(), l2g)
    assert np.array_equal(local.row_ptr.cpu().numpy(), rp)
    assert np.array_equal(local.col_idx.cpu().numpy(), ci)
    return local, l2g_d, (rp, ci, l2g, off, dl)


@pytest.mark.parametrize("fanout", [0, 3, 5, 100000])
def test_sampled_extraction_power_law(fanout):
    g = gg.chung_lu(40000, 15.0, 2.1, 81)
    pid = gg.bfs_partition(g, 8, 81)
    T = np.flatnonzero(pid == 0)
    _sampled_case(g, T, fanout, 0x5EED, "one of 8 parts")


def test_sampled_extraction_hub_outside_vertex_and_tiny_sets():
    n = 30000
    base = gg.erdos_renyi(n, 6.0, 82)
    rng = np.random.default_rng(82)
    T = np.sort(rng.choice(np.arange(1, n), 6000, replace=False))
    r = np.repeat(np.arange(n, dtype=np.int64), np.diff(base.row_ptr))
    c = base.col_idx.astype(np.int64)
    z = np.zeros(T.size, dtype=np.int64)
    g = gg.csr_from_edges(n, n, np.concatenate([r, z, T]), np.concatenate([c, T, z]))   # vertex 0 (outside) adjacent to every target
    local, l2g, (rp, ci, l2g_o, off, dl) = _sampled_case(g, T, 4, 7, "outside hub")
    k = int(np.searchsorted(l2g_o[len(T):], 0)) + len(T)
    assert l2g_o[k] == 0 and rp[k + 1] - rp[k] > 1024                     # a long reverse row
    _sampled_case(g, np.array([5]), 2, 1, "one target")


def test_training_step_after_sampling_and_extraction():
    """The sampled-partition chain at small size, all on the GPU: sample, extract, gather features, one bf16 training step."""
    import paper_2311_06837_amd as P
    n, dims, dtype = 40000, [64, 48, 48, 5], torch.bfloat16
    g = gg.chung_lu(n, 15.0, 2.1, 83)
    T = np.flatnonzero(gg.bfs_partition(g, 8, 83) == 0)
    local, l2g_d, (rp, ci, l2g, off, dl) = _sampled_case(g, T, 5, 0xABC, "model")
    n_local, L = l2g.size, 3
    params = gg.layer_weights(dims, True, 83)
    H0g = gg.features(n, dims[0], 83)
    y = gg.labels(len(T), dims[-1], 83)
    H0o = oracle.round_bf16(H0g.astype(np.float64))
    om = oracle.Model(rp, ci, np.arange(len(T), dtype=np.int32), "sage", params, bf16=True)
    loss_o = om.forward(H0o[l2g], y)
    grads_o = om.backward()
    H0d = torch.zeros(n_local, P.row_stride(dims[0], dtype), dtype=dtype, device="cuda")
    P.gnn_gather_rows(dev(H0g).to(dtype), l2g_d, dims[0], H0d)
    m = P.MaskedGNN(local, local, torch.arange(len(T), dtype=torch.int32, device="cuda"), "sage",
                    [{k: dev(v) for k, v in p.items()} for p in params], dtype=dtype, prefix_numbered=True,
                    transform_first=True)
    m.set_input(H0d)
    loss = m.step(dev(y))
    torch.cuda.synchronize()
    assert [int(x) for x in m.hop] == [0, len(T), n_local, n_local, n_local]      # dist is 0 or 1: every later ring is empty
    tol = TOL[dtype] * 2 * L
    assert abs(loss.item() - loss_o) <= tol * abs(loss_o), (loss.item(), loss_o)
    backward_at_the_oracles_point(m, om, dims, dtype, dev(y))     # same ReLU decisions on both sides, then element by element
    for l, gr in enumerate(grads_o):
        for k, want in gr.items():
            check(m.grads[l][k].double().cpu().numpy(), want, dtype, f"layer {l + 1} {k}", calls=L - l)


# ---- row-length classes ---------------------------------------------------------------------------------------

@pytest.mark.parametrize("L", [1, 4, 30])
def test_rows_at_the_edges_of_the_length_classes(L):
    """Rows of 64 / 65 (sixteen lanes / wavefront), 1024 / 1025 (wavefront / workgroup) and 2048 / 2049 entries (one step /
    two of the workgroup), each with neighbours at several distances."""
    n, lengths = 9000, [1, 16, 63, 64, 65, 1023, 1024, 1025, 2047, 2048, 2049, 6500]
    rng = np.random.default_rng(L)
    base = gg.random_directed(n, 1.2, 90 + L)
    r = np.repeat(np.arange(n, dtype=np.int64), np.diff(base.row_ptr))
    keep = r >= 200                                      # the first rows get the lengths in question
    rows, cols = [r[keep]], [base.col_idx[keep].astype(np.int64)]
    for k, ln in enumerate(lengths):
        rows.append(np.full(ln, 10 * k, dtype=np.int64))
        cols.append(np.sort(rng.choice(n, ln, replace=False)).astype(np.int64))
    g = gg.csr_from_edges(n, n, np.concatenate(rows), np.concatenate(cols))
    assert [int(g.degrees()[10 * k]) for k in range(len(lengths))] == lengths
    some = np.sort(rng.choice(np.arange(200, n), 5, replace=False))
    _extract_case(g, np.concatenate([[0, 40, 80], some]), L, "length classes, some of them targets")
    _extract_case(g, 10 * np.arange(len(lengths)), L, "length classes, all targets")


def test_reverse_rows_at_the_edges_of_the_length_classes_and_cut_by_the_capacity():
    """Outside vertices that 1, 2, 64, 65, 1024, 1025 and 3000 targets kept, and outputs with less room than entries: what
    fits is written in order, nothing beyond it."""
    import ctypes as C
    import paper_2311_06837_amd as P
    from paper_2311_06837_amd import binding as B
    n, nt, lengths = 8000, 4000, [1, 2, 15, 16, 17, 64, 65, 1024, 1025, 3000]
    rng = np.random.default_rng(91)
    a, b = [], []
    for k, ln in enumerate(lengths):                     # outside vertex nt + 7 k next to ln targets
        t = rng.choice(nt, ln, replace=False)
        a.append(t), b.append(np.full(ln, nt + 7 * k))
    inner = rng.integers(0, nt, size=(2, 6000))
    a, b = np.concatenate(a + [inner[0][inner[0] != inner[1]]]), np.concatenate(b + [inner[1][inner[0] != inner[1]]])
    g = gg.csr_from_edges(n, n, np.concatenate([a, b]).astype(np.int64), np.concatenate([b, a]).astype(np.int64))
    T = np.arange(nt)
    local, l2g_d, (rp, ci, l2g, off, dl) = _sampled_case(g, T, 100, 3, "reverse lengths")
    assert sorted(np.diff(rp)[nt:].tolist()) == lengths
    # the same fill pass into smaller outputs
    G = P.Graph.from_numpy(g.row_ptr, g.col_idx)
    Td = dev(T.astype(np.int32))
    srp, sci = P.gnn_sample_boundary(G, P.gnn_make_bitmap(Td, n), Td, 100, 3)
    gs = B.Graph(P.gnn_expand_row_ptr(n, Td, srp), sci.contiguous(), n_cols=n, sorted_columns=True)
    dist, ring, _, hop = P.gnn_build_active_sets(gs, Td, 1)
    n_local, nnz = int(hop[-1]), ci.size
    new_id = torch.empty(n, dtype=torch.int32, device="cuda")
    out_rp = torch.empty(n_local + 1, dtype=torch.int32, device="cuda")
    nnz_dev = torch.empty(1, dtype=torch.int64, device="cuda")
    common = (C.byref(G.c), C.byref(gs.c), B._ptr(ring), C.c_int32(n_local), B._ptr(dist), B._ptr(new_id), B._ptr(out_rp))
    B._with_ws(B.lib().gnn_extract_sampled_partition, common + (None, C.c_int64(0), B._ptr(nnz_dev), None), (B._stream(),), None)
    starts = [int(rp[j]) for j in range(nt, n_local)]
    for cap in sorted({0, 1, int(rp[nt]) - 1, nnz - 1, nnz} | {s + d for s in starts for d in (1, 40)}):
        if cap > nnz:
            continue
        out = torch.full((nnz,), -7, dtype=torch.int32, device="cuda")
        B._with_ws(B.lib().gnn_extract_sampled_partition, common + (B._ptr(out), C.c_int64(cap), B._ptr(nnz_dev), None), (B._stream(),), None)
        got = out.cpu().numpy()
        assert np.array_equal(got[:cap], ci[:cap]) and (got[cap:] == -7).all(), cap


def _multigraph(n, a, b, times):
    """Symmetric CSR whose edges (a[i], b[i]) appear times[i] times in both directions, columns ascending."""
    a, b = np.repeat(a, times), np.repeat(b, times)
    r, c = np.concatenate([a, b]).astype(np.int64), np.concatenate([b, a]).astype(np.int64)
    order = np.lexsort((c, r))
    rp = np.zeros(n + 1, dtype=np.int32)
    rp[1:] = np.cumsum(np.bincount(r, minlength=n))
    return gg.CSR(n, n, rp, c[order].astype(np.int32))


@pytest.mark.parametrize("whole", [True, False])
def test_reverse_rows_of_kept_rows_that_repeat_a_column(whole):
    """Kept rows of the caller's own, in which columns repeat (a repeated column counts as often as it appears): reverse rows of
    every length class, ascending, with every target as often as its kept row holds the vertex; `whole` False: some copies
    of an edge are kept and others not.  Then the same into outputs that are too small."""
    import ctypes as C
    import paper_2311_06837_amd as P
    from paper_2311_06837_amd import binding as B
    n, nt = 9000, 4000
    rng = np.random.default_rng(17 + whole)
    a, b = [], []
    for k, ln in enumerate([1, 2, 3, 10, 30, 33, 400, 600, 1500, 3900]):    # outside vertex nt + 5 k next to ln targets
        a.append(rng.choice(nt, ln, replace=False)), b.append(np.full(ln, nt + 5 * k))
    a, b = np.concatenate(a), np.concatenate(b)
    g = _multigraph(n, a, b, rng.integers(1, 4, a.size))
    T = np.arange(nt, dtype=np.int32)
    keep = np.ones(g.nnz, dtype=bool) if whole else rng.random(g.nnz) < 0.7
    row = np.repeat(np.arange(n), np.diff(g.row_ptr))
    keep &= row < nt
    srp = np.zeros(nt + 1, dtype=np.int32)
    srp[1:] = np.cumsum(np.bincount(row[keep], minlength=nt)[:nt])
    sci = g.col_idx[keep]
    rp, ci, l2g, off, dl = oracle.extract_sampled(n, T, srp, sci)
    lens = np.diff(rp)[nt:]
    assert lens.min() < 10 and ((lens > 64) & (lens <= 1024)).any() and (lens > 1024).sum() >= 2
    G, Td = P.Graph.from_numpy(g.row_ptr, g.col_idx), dev(T)
    local, l2g_d, hop = P.gnn_extract_sampled_partition(G, Td, dev(srp), dev(sci))
    assert list(hop) == list(off) and np.array_equal(l2g_d.cpu().numpy(), l2g)
    assert np.array_equal(local.row_ptr.cpu().numpy(), rp)
    assert np.array_equal(local.col_idx.cpu().numpy(), ci)
    gs = B.Graph(P.gnn_expand_row_ptr(n, Td, dev(srp)), dev(sci), n_cols=n, sorted_columns=True)
    dist, ring, _, hop = P.gnn_build_active_sets(gs, Td, 1)
    new_id = torch.empty(n, dtype=torch.int32, device="cuda")
    out_rp = torch.empty(len(l2g) + 1, dtype=torch.int32, device="cuda")
    nnz_dev = torch.empty(1, dtype=torch.int64, device="cuda")
    common = (C.byref(G.c), C.byref(gs.c), B._ptr(ring), len(l2g), B._ptr(dist), B._ptr(new_id), B._ptr(out_rp))
    B._with_ws(B.lib().gnn_extract_sampled_partition, common + (None, 0, B._ptr(nnz_dev), None), (B._stream(),), None)
    for cap in sorted({int(rp[j]) + d for j in range(nt, len(l2g)) for d in (1, 2, 37)}):
        if cap > ci.size:
            continue
        out = torch.full((ci.size,), -7, dtype=torch.int32, device="cuda")
        B._with_ws(B.lib().gnn_extract_sampled_partition, common + (B._ptr(out), cap, B._ptr(nnz_dev), None), (B._stream(),), None)
        got = out.cpu().numpy()
        assert np.array_equal(got[:cap], ci[:cap]) and (got[cap:] == -7).all(), cap


@pytest.mark.parametrize("all_reached", [False, True])
def test_more_vertices_than_a_limited_grid_has_threads(all_reached):
    """2^28 + 5000 vertices, edges between the last 4000: extraction of the last vertices, and of everything."""
    import paper_2311_06837_amd as P
    n, m = 2 ** 28 + 5000, 4000
    rp = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
    rp[n - m + 1:] = torch.arange(1, m + 1, dtype=torch.int32, device="cuda")
    ci = torch.arange(n - m + 1, n + 1, dtype=torch.int32, device="cuda")
    ci[-1] = n - m                                               # a cycle through the last m vertices
    g = P.Graph(rp, ci, sorted_columns=True)
    T = torch.arange(0 if all_reached else n - 3000, n, dtype=torch.int32, device="cuda")
    dist, ring, _, hop = P.gnn_build_active_sets(g, T, 1)
    n_local = n if all_reached else 3001
    assert hop[-1] == n_local
    local, new_id = P.gnn_extract_partition(g, ring, n_local, dist, 1)
    if all_reached:
        assert torch.equal(local.row_ptr, rp) and torch.equal(local.col_idx, ci)
        assert torch.equal(new_id, torch.arange(n, dtype=torch.int32, device="cuda"))
        del local, new_id, dist, ring
        assert torch.equal(P.gnn_expand_row_ptr(n, T, rp), rp)
    else:       # the targets in order, then vertex n - m, the last target's neighbour, whose own neighbour is out of reach
        assert torch.equal(local.row_ptr, torch.arange(3002, dtype=torch.int32, device="cuda").clamp(max=3000))
        assert torch.equal(local.col_idx, torch.arange(1, 3001, dtype=torch.int32, device="cuda"))


@pytest.mark.parametrize("n", [1, 1023, 8192, 8193, 9216, 9217, 10240, 10241, 1 << 23, (1 << 23) + 1])
def test_offsets_across_the_forms_of_the_scan(n):
    """One block up to 10 240 counts, blocks that add up the sums before their own up to 8192 blocks of 1024, a launch for the sums above."""
    import paper_2311_06837_amd as P
    print(f"offsets of {n} counts", flush=True)
    ids = torch.arange(0, n, 3, dtype=torch.int32, device="cuda")
    gen = torch.Generator(device="cuda").manual_seed(n)
    length = torch.randint(0, 200, (ids.numel(),), device="cuda", generator=gen)
    rp = torch.zeros(ids.numel() + 1, dtype=torch.int32, device="cuda")
    rp[1:] = torch.cumsum(length, 0)
    full = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    full[1 + ids.long()] = length
    assert torch.equal(P.gnn_expand_row_ptr(n, ids, rp).long(), torch.cumsum(full, 0))
