"""GPU parity: gnn_build_active_sets against the oracle, bit-exact (section 6, steps 1 and 4)."""
import numpy as np
import pytest
import torch

import graphgen as gg
import oracle
from gpu_util import dev

pytestmark = pytest.mark.gpu


def _run(g, targets, L, with_transpose):
    import paper_2311_06837_amd as P
    G = P.Graph.from_numpy(g.row_ptr, g.col_idx)
    GT = None
    if with_transpose:
        t = gg.transpose(g)
        GT = P.Graph.from_numpy(t.row_ptr, t.col_idx)
    t = dev(np.asarray(targets, dtype=np.int32))
    dist, ring, off, hop = P.gnn_build_active_sets(G, t, L, gt=GT)
    torch.cuda.synchronize()
    return dist.cpu().numpy(), ring.cpu().numpy(), off.cpu().numpy(), hop


def _compare(g, targets, L):
    """Both forms of the call - every level from the frontier, and with the transposed graph (levels may then run from
    the unreached vertices) - against the oracle's plain breadth-first levels."""
    valid = np.asarray(targets, dtype=np.int64)
    valid = valid[(valid >= 0) & (valid < g.n_rows)]
    od, oring, ooff = oracle.active_sets(g.row_ptr, g.col_idx, valid.astype(np.int32), L)
    for with_transpose in (False, True):
        print(f"active sets: n={g.n_rows} nnz={g.nnz} |T|={len(targets)} L={L} transposed graph given: {with_transpose}", flush=True)
        dist, ring, off, hop = _run(g, targets, L, with_transpose)
        assert np.array_equal(off, ooff) and list(hop) == list(ooff)
        assert np.array_equal(dist, od)
        assert np.array_equal(ring[: ooff[-1]], oring)


def _sym(n, und):
    r = np.array([a for a, b in und] + [b for a, b in und], dtype=np.int64)
    c = np.array([b for a, b in und] + [a for a, b in und], dtype=np.int64)
    return gg.csr_from_edges(n, n, r, c)


def test_closed_form_graphs():
    _compare(_sym(21, [(i, i + 1) for i in range(20)]), [10], 4)
    _compare(_sym(9, [(0, i) for i in range(1, 9)]), [0], 3)            # empty late rings
    _compare(_sym(8, [(0, 1), (1, 2), (2, 3), (4, 5), (5, 6), (6, 7)]), [0], 5)   # unreachable part
    _compare(_sym(12, [(i, j) for i in range(12) for j in range(i + 1, 12)]), [2, 5], 3)


@pytest.mark.parametrize("seed", [0, 1])
def test_random_graphs_directed_and_symmetric(seed):
    rng = np.random.default_rng(seed)
    g = gg.erdos_renyi(20000, 6.0, seed)
    _compare(g, rng.choice(20000, 300, replace=False), 3)
    d = gg.random_directed(30011, 3.0, seed)                              # ragged bitmap tail
    _compare(d, rng.choice(30011, 500, replace=False), 5)


def test_power_law_with_hub_rows():
    g = gg.chung_lu(60000, 60.0, 2.1, 7)                                  # max degree ~ 1900
    assert g.degrees().max() > 1024
    _compare(g, np.arange(0, 60000, 97), 2)
    big = gg.chung_lu(20000, 1500.0, 2.1, 8)                              # rows above the 4096 hub split
    assert big.degrees().max() > 4096
    _compare(big, np.arange(0, 20000, 501), 2)


def test_edge_cases():
    g = gg.erdos_renyi(500, 4.0, 3)
    _compare(g, [], 2)                                                    # no targets
    _compare(g, [7, 7, 7, 3, 3], 2)                                       # repeated targets
    _compare(g, [5, -1, 500, 10**6, 9], 2)                                # out-of-range ids are ignored
    _compare(g, np.arange(500), 1)                                        # everything is a target
    empty = gg.CSR(64, 64, np.zeros(65, dtype=np.int32), np.zeros(0, dtype=np.int32))
    _compare(empty, [1, 2, 3], 3)                                         # no edges
    _compare(g, [0], 40)                                                  # far more levels than the diameter


def test_deep_shrinking_sets_like_cfg3():
    w = gg.make_workload("cfg3", scale=0.03)
    p = w.partition
    _compare(p.graph, p.targets, w.n_layers)


def test_levels_that_run_from_the_unreached_vertices():
    """Graphs on which the direction switch picks the pull form: a frontier that is most of the graph (dense power
    law), directed edges (the transposed rows differ from the rows), a long transposed row that is still unreached
    when the switch happens (its own workgroup), and unreached vertices that no frontier vertex reaches."""
    g = gg.chung_lu(50000, 200.0, 2.1, 17)                                # ring 1 is most of the graph
    _compare(g, np.arange(0, 50000, 9), 3)
    d = gg.random_directed(40000, 40.0, 5)
    _compare(d, np.arange(0, 40000, 7), 4)
    # Long transposed rows that are still unreached when a level pulls (a workgroup each): the centre of a star in a
    # component the targets do not touch (no entry is in the frontier), and a vertex that 3000 vertices of the dense
    # part aggregate from while it aggregates from nobody (reached by the pull, through one of them).
    na = 30000
    dense = gg.chung_lu(na, 100.0, 2.1, 3)
    centre, leaves = na, np.arange(na + 1, na + 5001)
    h = na + 5001
    n = h + 1
    fans = np.arange(1, na, 10)[:3000]                                    # no target among them (targets are multiples of 10)
    rows = np.concatenate([np.repeat(np.arange(na), np.diff(dense.row_ptr)), np.full(5000, centre), leaves, fans])
    cols = np.concatenate([dense.col_idx.astype(np.int64), leaves, np.full(5000, centre), np.full(3000, h)])
    g2 = gg.csr_from_edges(n, n, rows, cols)
    assert np.diff(gg.transpose(g2).row_ptr)[[centre, h]].min() >= 3000
    _compare(g2, np.arange(0, na, 10), 3)
    iso = gg.csr_from_edges(n, n, np.repeat(np.arange(n // 2), 60),
                            np.random.default_rng(0).integers(0, n // 2, 60 * (n // 2)))   # half the graph is unreachable
    _compare(iso, np.arange(0, n // 2, 5), 3)


# ---- graphs of many compaction blocks (8192 vertices each) ---------------------------------------------------------

def _chain(n):
    """v -> v + 1, and its transpose; the last vertex has no neighbour."""
    import paper_2311_06837_amd as P
    at = torch.arange(n + 1, dtype=torch.int64, device="cuda")
    g = P.Graph(at.clamp(max=n - 1).int(), torch.arange(1, n, dtype=torch.int32, device="cuda"))
    gt = P.Graph((at - 1).clamp(min=0).int(), torch.arange(n - 1, dtype=torch.int32, device="cuda"))
    return g, gt


@pytest.mark.parametrize("n", [8192 * 256, 8192 * 256 + 1, 8192 * 2048, 8192 * 2048 + 1, 20_000_003])
def test_sets_of_graphs_with_many_blocks(n):
    """On both sides of 256 and of 2048 blocks: rings of a thousandth of the vertices, a dense stretch beside them, and nearly
    all vertices (a level from the unreached ones), with and without the transposed graph."""
    import paper_2311_06837_amd as P
    g, gt = _chain(n)
    sparse = torch.arange(7, n, 1000, device="cuda")
    dense = torch.unique(torch.cat([sparse, torch.arange(n // 2, n // 2 + 20_000, device="cuda"), torch.arange(n - 40, n - 3, 5, device="cuda")]))
    most = torch.arange(n, device="cuda")
    most = most[(most % 100 < 96) | (most < n // 2)]
    for name, T in (("sparse", sparse), ("dense", dense), ("most", most)):
        L = 2
        want = torch.full((n,), -1, dtype=torch.int32, device="cuda")
        for d in range(L, -1, -1):
            want[T[T < n - d] + d] = d
        for t in (None, gt):
            print(f"sets: chain of {n}, {name}, {'with' if t else 'without'} transpose", flush=True)
            dist, ring, _, hop = P.gnn_build_active_sets(g, T.int(), L, gt=t)
            assert torch.equal(dist, want)
            order = torch.cat([torch.nonzero(want == d).reshape(-1) for d in range(L + 1)]).int()
            assert hop == [0] + torch.cumsum(torch.stack([(want == d).sum() for d in range(L + 1)]), 0).tolist()
            assert torch.equal(ring[: int(hop[-1])], order)
        d, r, _, hop = P.gnn_eas_traverse(g, T.int(), 1, 1, "hash", 3)      # a vertex has one neighbour: the same sets
        assert torch.equal(d, torch.where(want > 1, -1, want))


def test_cost_of_the_direction_switch_in_large_graphs():
    """What the transposed graph adds to a construction (the sums that choose the direction) stays below the construction
    itself: sums that all workgroups add to one address were twice that at this size."""
    import paper_2311_06837_amd as P
    n = 100_000_000
    g, gt = _chain(n)
    T = torch.arange(0, n, 1000, dtype=torch.int32, device="cuda")
    ws = P.Workspace()

    def time_us(t):
        times = []
        for _ in range(4):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            P.gnn_build_active_sets(g, T, 3, sync=False, ws=ws, gt=t)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b) * 1e3)
        return min(times)
    assert time_us(gt) < 2 * time_us(None)


@pytest.mark.parametrize("n,nnz", [(32768, 131072), (32768, 131073), (32769, 100_000), (31, 40), (1025, 131072), (4097, 60_000)])
def test_sets_of_small_graphs_around_the_one_launch_limit(n, nnz):
    """One workgroup builds the sets of graphs of up to 32 768 vertices and 131 072 entries: rows without entries, a hub,
    repeated entries, targets out of range, more levels than rings, more than 4096 vertices in a ring."""
    rng = np.random.default_rng(nnz)
    rows = np.sort(np.where(rng.random(nnz) < 0.2, 3 % n, rng.integers(0, max(1, n * 3 // 4), nnz)))
    cols = rng.integers(0, n, nnz)
    row_ptr = np.zeros(n + 1, np.int32)
    row_ptr[1:] = np.cumsum(np.bincount(rows, minlength=n))
    import paper_2311_06837_amd as P
    G = P.Graph(dev(row_ptr), dev(cols.astype(np.int32)))
    for targets in ([n - 1, 0, 0, -1, n], rng.integers(0, n, max(1, n // 3)), []):
        for L in (1, 3, 12):
            targets = np.asarray(targets, dtype=np.int32)
            valid = targets[(targets >= 0) & (targets < n)]
            od, oring, ooff = oracle.active_sets(row_ptr, cols.astype(np.int32), valid, L)
            dist, ring, off, hop = P.gnn_build_active_sets(G, dev(targets), L)
            assert list(hop) == list(ooff) and np.array_equal(off.cpu().numpy(), ooff)
            assert np.array_equal(dist.cpu().numpy(), od) and np.array_equal(ring.cpu().numpy()[: ooff[-1]], oring)


@pytest.mark.parametrize("deg", [1, 4])
def test_sets_of_a_small_graph_whose_every_vertex_has_entries(deg):
    """Whole steps of 4096 rows with entries, at both limits of the one-launch form: the two counts that share an integer."""
    import paper_2311_06837_amd as P
    n = 32_768
    cols = ((np.arange(n)[:, None] + 1 + np.arange(deg) * 5000) % n).astype(np.int32)
    cols.sort(axis=1)
    row_ptr = (np.arange(n + 1) * deg).astype(np.int32)
    G = P.Graph(dev(row_ptr), dev(cols.reshape(-1)))
    for targets in (np.arange(n, dtype=np.int32), np.arange(0, n, 3, dtype=np.int32), np.arange(4096, dtype=np.int32)):
        od, oring, ooff = oracle.active_sets(row_ptr, cols.reshape(-1), targets, 6)
        dist, ring, off, hop = P.gnn_build_active_sets(G, dev(targets), 6)
        assert list(hop) == list(ooff) and np.array_equal(dist.cpu().numpy(), od)
        assert np.array_equal(ring.cpu().numpy()[: ooff[-1]], oring)


@pytest.mark.parametrize("deg,L", [(1, 2), (2, 2), (3, 4), (3, 5)])
def test_sets_on_either_side_of_the_small_graphs_rule(deg, L):
    """nnz + 3 n <= 168 000, or five levels: 32 000 vertices of degree 2 are taken by one launch, of degree 3 from five levels on."""
    import paper_2311_06837_amd as P
    n = 32_000
    cols = np.sort((np.arange(n)[:, None] + 1 + np.arange(deg) * 5000) % n, axis=1).astype(np.int32)
    row_ptr = (np.arange(n + 1) * deg).astype(np.int32)
    G = P.Graph(dev(row_ptr), dev(cols.reshape(-1)))
    targets = np.arange(0, n, 7, dtype=np.int32)
    od, oring, ooff = oracle.active_sets(row_ptr, cols.reshape(-1), targets, L)
    dist, ring, off, hop = P.gnn_build_active_sets(G, dev(targets), L, gt=None)
    assert list(hop) == list(ooff) and np.array_equal(dist.cpu().numpy(), od)
    assert np.array_equal(ring.cpu().numpy()[: ooff[-1]], oring)


def test_a_hub_in_a_small_graph_costs_no_more_than_in_a_larger_one():
    """32 000 vertices around one hub, 96 000 entries: not for one workgroup (82 us where the form with a launch per part of a level
    takes 42).  32 800 vertices take that form by their number."""
    import paper_2311_06837_amd as P

    def time_us(n):
        i = np.arange(n, dtype=np.int64)
        keys = np.unique(np.concatenate([i[1:] * n, i[1:], i * n + (i * 7 + 1) % n]))
        row_ptr = np.searchsorted(keys, np.arange(n + 1, dtype=np.int64) * n).astype(np.int32)
        G = P.Graph(dev(row_ptr), dev((keys % n).astype(np.int32)))
        T, ws, times = dev(np.array([0, n // 2], np.int32)), P.Workspace(), []
        for _ in range(6):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(20):
                P.gnn_build_active_sets(G, T, 3, sync=False, ws=ws)
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b) * 50)
        return min(times)
    assert time_us(32_000) < 1.4 * time_us(32_800)


@pytest.mark.parametrize("n_targets,n_left", [(8193, 4096), (8192, 4096), (20_000, 4097), (20_000, 31), (3, 1), (2, 1), (70, 0)])
def test_small_graphs_whose_last_vertices_look_for_themselves(n_targets, n_left):
    """One launch with the transposed graph: a level behind which few vertices are left starts from those (at most 4096, fewer than half
    of the ring).  Some are reached at once, some by the others one level on, one has many entries, some have none."""
    rng = np.random.default_rng(n_left)
    n = n_targets + n_left
    left = np.arange(n_targets, n)
    first, second = left[: n_left // 2], left[n_left // 2: n_left - n_left // 4]      # the rest is never reached
    rows = [rng.integers(0, n_targets, first.size), rng.integers(0, n_targets, n_targets)]
    cols = [first, rng.integers(0, n_targets, n_targets)]
    if first.size:
        rows += [first[rng.integers(0, first.size, second.size)], rng.integers(0, n_targets, 3000)]
        cols += [second, np.full(3000, first[0])]
    rows += [second, left]
    cols += [rng.integers(0, n_targets, second.size), left]
    g = gg.csr_from_edges(n, n, np.concatenate(rows).astype(np.int64), np.concatenate(cols).astype(np.int64))
    for L in (1, 2, 4):
        _compare(g, rng.permutation(n_targets).astype(np.int32), L)


def test_last_vertices_that_hold_the_entries_do_not_look_for_themselves():
    """12 000 vertices, of which 3900 hold all entries among themselves and are never reached: nothing to walk from the ring, 100 000
    entries from the last vertices.  Knowing the transposed graph must not cost (17 us without it, 33 from the last vertices)."""
    import paper_2311_06837_amd as P
    n, n_left = 12_000, 3900
    rng = np.random.default_rng(4)
    a, b = rng.integers(n - n_left, n, (2, n_left * 13))
    g = gg.csr_from_edges(n, n, np.concatenate([a, b]).astype(np.int64), np.concatenate([b, a]).astype(np.int64))
    targets = np.arange(n - n_left, dtype=np.int32)
    G = P.Graph(dev(g.row_ptr), dev(g.col_idx))
    T, ws = dev(targets), P.Workspace()

    def time_us(gt):
        times = []
        for _ in range(6):
            x, y = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            x.record()
            for _ in range(20):
                P.gnn_build_active_sets(G, T, 2, sync=False, ws=ws, gt=gt)
            y.record()
            y.synchronize()
            times.append(x.elapsed_time(y) * 50)
        return min(times)
    od, oring, ooff = oracle.active_sets(g.row_ptr, g.col_idx, targets, 2)
    dist, ring, off, hop = P.gnn_build_active_sets(G, T, 2, gt=G)
    assert list(hop) == list(ooff) and np.array_equal(dist.cpu().numpy(), od)
    with_gt, without = time_us(G), time_us(None)
    print(with_gt, without, flush=True)
    assert with_gt < 1.4 * without
