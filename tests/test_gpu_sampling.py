"""GPU parity: gnn_sample_boundary and gnn_make_bitmap against the oracle, bit-exact
(section 5.3 with the seeded hash rule)."""
import numpy as np
import pytest
import torch

import graphgen as gg
import oracle
from gpu_util import dev

pytestmark = pytest.mark.gpu


def _compare(g, T, fanout, seed):
    import paper_2311_06837_amd as P
    print(f"sampling: n={g.n_rows} nnz={g.nnz} |T|={len(T)} f={fanout} seed={seed:#x}", flush=True)
    G = P.Graph.from_numpy(g.row_ptr, g.col_idx)
    Td = dev(np.asarray(T, dtype=np.int32))
    bits = P.gnn_make_bitmap(Td, g.n_rows)
    rp, ci = P.gnn_sample_boundary(G, bits, Td, fanout, seed)
    torch.cuda.synchronize()
    is_t = np.zeros(g.n_rows, dtype=np.uint8)
    is_t[T] = 1
    want_bits = np.packbits(is_t.astype(bool), bitorder="little")
    got_bits = bits.cpu().numpy().view(np.uint8)[: want_bits.size]
    assert np.array_equal(got_bits, want_bits)
    orp, oci = oracle.sample_boundary(g.row_ptr, g.col_idx, is_t, T, fanout, seed)
    assert np.array_equal(rp.cpu().numpy(), orp)
    assert np.array_equal(ci.cpu().numpy(), oci)


@pytest.mark.parametrize("fanout", [0, 1, 5, 15])
def test_power_law_partition(fanout):
    g = gg.chung_lu(40000, 15.0, 2.1, 31)
    pid = gg.bfs_partition(g, 8, 31)
    T = np.flatnonzero(pid == 0).astype(np.int32)
    _compare(g, T, fanout, 0x5EED0004)


def test_hub_rows_and_large_fanout_and_seed_range():
    g = gg.chung_lu(8000, 300.0, 2.1, 32)                 # rows far longer than one wavefront
    assert g.degrees().max() > 1200
    T = np.arange(0, 8000, 3).astype(np.int32)
    _compare(g, T, 5, 1)
    _compare(g, T, 70, 2**64 - 1)                         # fanout above the wavefront width; seed + hop wraps
    _compare(g, T, int(g.degrees().max()), 3)             # keeps everything


def test_unsorted_targets_and_edge_cases():
    g = gg.erdos_renyi(3000, 8.0, 33)
    rng = np.random.default_rng(0)
    T = rng.permutation(3000)[:1025].astype(np.int32)     # ragged count, arbitrary order
    _compare(g, T, 2, 9)
    _compare(g, np.zeros(0, dtype=np.int32), 2, 9)        # no targets
    _compare(g, np.arange(3000, dtype=np.int32), 2, 9)    # no outside neighbours at all


def test_row_lengths_around_the_sixteen_lane_limit():
    """Rows of 63 / 64 / 65 entries (the last one leaves its sixteen lanes for a workgroup), of 1023 / 1024 / 1025 (one step
    of that workgroup's sweep, then two) and an empty one, targets and outside vertices mixed in every row."""
    rng = np.random.default_rng(35)
    n = 5000
    lens = [63, 64, 65, 0, 1023, 1024, 1025, 1, 256, 257, 4097]
    rows, cols = [], []
    for r, ln in enumerate(lens):
        c = rng.choice(n, size=ln, replace=False)
        rows.append(np.full(ln, r, dtype=np.int64))
        cols.append(c.astype(np.int64))
    g = gg.csr_from_edges(n, n, np.concatenate(rows), np.concatenate(cols))
    assert list(g.degrees()[: len(lens)]) == lens
    T = np.concatenate([np.arange(len(lens)), np.arange(100, n, 2)]).astype(np.int32)   # about half of every row is inside
    for fanout in (0, 1, 3, 40, 150, 250, 600):    # the long rows: from the listed keys up to 150, then by sweeps over the row
        _compare(g, T, fanout, 0xABCDEF)


def _mix64(x):
    with np.errstate(over="ignore"):
        x = x + np.uint64(0x9E3779B97F4A7C15)
        x = (x ^ (x >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        x = (x ^ (x >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        return x ^ (x >> np.uint64(31))


@pytest.mark.parametrize("length", [64, 65, 256, 257, 1024])
def test_rows_in_which_the_upper_halves_of_two_keys_are_equal(length):
    """The selection compares upper halves and falls back to whole pairs where the k-th is not alone with its half: rows built
    around two outside neighbours whose keys share it, kept both, one of them, or neither."""
    n, seed, v = 1_500_000, 77, 5
    keys = _mix64(_mix64(_mix64(np.uint64(seed + 1)) ^ np.uint64(v)) ^ np.arange(n, dtype=np.uint64))
    assert int(keys[123]) == oracle.edge_key(seed, v, 123, 1)
    order = np.argsort(keys)
    half = keys[order] >> np.uint64(32)
    at = np.flatnonzero(half[1:] == half[:-1])
    at = int(at[at > length][0])                               # the pair is order[at], order[at + 1]
    for k in (1, 2, 10):
        for before in sorted({max(k - 1, 0), max(k - 2, 0), k}):
            low = order[np.random.default_rng(before).choice(at, before, replace=False)]
            high = order[at + 2:][np.random.default_rng(k).choice(n - at - 2, length - before - 2, replace=False)]
            cols = np.sort(np.concatenate([low, order[at: at + 2], high])).astype(np.int32)
            row_ptr = np.zeros(n + 1, dtype=np.int32)
            row_ptr[v + 1:] = length
            inner = [int(c) for c in high[:3] if c != v]
            _compare(gg.CSR(n, n, row_ptr, cols), np.array([v] + inner, dtype=np.int32), k, seed)


def test_more_targets_than_a_launch_takes_at_a_time():
    """Every lane group takes several rows, one after the other, of every length class."""
    g = gg.chung_lu(150_000, 12.0, 2.1, 36)
    _compare(g, np.arange(0, 150_000, 2).astype(np.int32), 3, 21)


@pytest.mark.parametrize("n", [1_000_003, 3_000_001])
def test_queues_of_millions_of_medium_rows(n):
    """Rows of 100 entries all go to the queue of the medium rows.  A workgroup appends a whole list of them with one atomic however
    many there are: three times the rows take about three times as long (fifteen, where the lists overflow)."""
    import torch
    import paper_2311_06837_amd as P
    deg = 100

    def graph(rows):
        step = rows // deg
        cols = torch.arange(deg, device="cuda")[None] * step + torch.randint(step, (rows, deg), device="cuda")      # ascending, distinct
        return P.Graph((torch.arange(rows + 1, device="cuda") * deg).int(), cols.int().reshape(-1), sorted_columns=True)

    def calls(g):
        ids = torch.arange(g.n_rows, device="cuda").int()
        bits = P.gnn_make_bitmap(ids[:-1], g.n_rows)
        dist = torch.zeros_like(ids)
        ws = P.Workspace()
        both = (lambda: P.gnn_sample_boundary(g, bits, ids, 3, 7, ws=ws),
                lambda: P.gnn_extract_partition(g, ids, g.n_rows, dist, 1, ws=ws))
        out, us = [], []
        for f in both:
            out.append(f())
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(3):
                f()
            b.record()
            b.synchronize()
            us.append(a.elapsed_time(b) / 3e-3)
        return out, us
    g = graph(n)
    (sampled, (local, _)), us = calls(g)
    for got in (sampled, (local.row_ptr, local.col_idx)):        # at most one neighbour of a row lies outside: all are kept
        assert torch.equal(got[0], g.row_ptr) and torch.equal(got[1], g.col_idx)
    del sampled, local
    few = 500_000
    _, us_few = calls(graph(few))
    print(n, us, us_few, flush=True)
    assert all(t <= 2.0 * n / few * t_few for t, t_few in zip(us, us_few))
