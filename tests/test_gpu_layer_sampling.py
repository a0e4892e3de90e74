"""GPU parity of layer-wise sampling as per-layer masking (section 5.2): gnn_layer_edge_mask and
gnn_transpose_edge_mask bit-exact against the oracle, the aggregation calls through gnn_csr.edge_keep against the
oracle's masked aggregation (fp32 1e-4, bf16 2e-2), and one training step of the model with per-layer masks."""
import numpy as np
import pytest
import torch

import graphgen as gg
import oracle
from gpu_util import TOL, as_stored, backward_at_the_oracles_point, check, dev, host64, padded

pytestmark = pytest.mark.gpu

M64 = (1 << 64) - 1
SENT = 4321.0


def _bits(words: torch.Tensor, nnz: int) -> np.ndarray:
    w = words.cpu().numpy().view(np.uint32)
    return ((w[np.arange(nnz) >> 5] >> (np.arange(nnz) & 31).astype(np.uint32)) & 1).astype(np.uint8)


def _pack(keep: np.ndarray) -> torch.Tensor:
    nnz = keep.shape[0]
    w = np.zeros(max((nnz + 31) // 32, 1), dtype=np.uint32)
    np.bitwise_or.at(w, np.arange(nnz) >> 5, keep.astype(np.uint32) << (np.arange(nnz) & 31).astype(np.uint32))
    return torch.from_numpy(w.view(np.int32)).cuda()


def _mask_case(g, rows, rule, par, layer, seed):
    import paper_2311_06837_amd as P
    print(f"layer mask: n={g.n_rows} nnz={g.nnz} rows={'all' if rows is None else len(rows)} rule={rule} par={par} layer={layer}", flush=True)
    G = P.Graph.from_numpy(g.row_ptr, g.col_idx)
    n_active = g.n_rows if rows is None else len(rows)
    kw = dict(fanout=par) if rule == "fanout" else dict(threshold=par)
    keep, kept_len = P.gnn_layer_edge_mask(G, dev(np.asarray(rows, dtype=np.int32)) if rows is not None and len(rows) else None,
                                           n_active, rule, layer, seed, **kw)
    torch.cuda.synchronize()
    okeep, olen = oracle.layer_edge_mask(g.row_ptr, g.col_idx, None if rows is None else np.asarray(rows, dtype=np.int32), rule, layer, seed, **kw)
    assert np.array_equal(_bits(keep, g.nnz), okeep)
    assert np.array_equal(kept_len.cpu().numpy(), olen)
    return G, keep, okeep


@pytest.mark.parametrize("rule,par", [("threshold", oracle.keep_threshold(0.5)), ("threshold", M64), ("threshold", 0),
                                      ("fanout", 1), ("fanout", 5), ("fanout", 25), ("fanout", 0), ("fanout", 10**6)])
def test_masks_power_law_graph(rule, par):
    g = gg.chung_lu(30011, 22.0, 2.1, 3)
    rng = np.random.default_rng(5)
    _mask_case(g, None, rule, par, 1, 42)
    _mask_case(g, np.sort(rng.choice(30011, 9000, replace=False)), rule, par, 3, 43)
    _mask_case(g, rng.permutation(30011)[:777], rule, par, 2, 2 ** 63 + 5)          # unsorted list, large seed


def test_masks_hub_rows_empty_rows_and_nothing_listed():
    g = gg.chung_lu(12000, 150.0, 2.1, 12)
    assert g.degrees().max() > 1024
    _mask_case(g, None, "fanout", 15, 1, 1)
    _mask_case(g, None, "threshold", oracle.keep_threshold(0.1), 2, 1)
    big = gg.chung_lu(20000, 1500.0, 2.1, 8)                  # rows with several times the entries a wavefront lists in LDS
    assert big.degrees().max() > 4096
    _mask_case(big, None, "fanout", 30, 1, 2)
    _mask_case(big, np.arange(0, 20000, 7), "fanout", 1, 2, 3)
    _mask_case(big, np.arange(0, 20000, 3), "fanout", 990, 1, 4)     # rows of up to 1024 entries: rounds over registers, longer ones:
    _mask_case(big, np.arange(0, 20000, 3), "fanout", 960, 1, 5)     # the wide list
    d = gg.random_directed(5000, 1.5, 13)
    assert (d.degrees() == 0).any()
    _mask_case(d, None, "fanout", 2, 1, 9)
    _mask_case(d, [], "fanout", 2, 1, 9)
    empty = gg.CSR(40, 40, np.zeros(41, dtype=np.int32), np.zeros(0, dtype=np.int32))
    _mask_case(empty, None, "threshold", M64, 1, 0)


def _rows_of(lengths, n_cols, seed):
    rng = np.random.default_rng(seed)
    cols = [np.sort(rng.choice(n_cols, ln, replace=False)).astype(np.int32) for ln in lengths]
    rp = np.zeros(len(lengths) + 1, dtype=np.int32)
    rp[1:] = np.cumsum(lengths)
    return gg.CSR(len(lengths), n_cols, rp, np.concatenate(cols))


@pytest.mark.parametrize("fanout", [1, 45, 46, 64, 65, 100, 144, 145, 500, 1023, 1024, 1025, 2999, 4624, 4625, 9000])
def test_fanouts_around_the_limits_of_the_lists(fanout):
    """Rows on both sides of what sixteen lanes (64) and registers (1024) hold, and longer ones, at fanouts on both sides of
    where the list of a long row starts above nothing (46), gets wide (145) and is given up (4625): bits, kept lengths and
    threshold pairs."""
    import paper_2311_06837_amd as P
    g = _rows_of([20, 64, 65, 900, 1024, 1025, 1300, 3000, 5000, 12000, 40000] * 2, 50000, fanout)
    G, keep, okeep = _mask_case(g, None, "fanout", fanout, 1, 77)
    _, kept_len, tk, tu = P.gnn_layer_edge_mask(G, None, g.n_rows, "fanout", 1, 77, fanout=fanout, with_thresholds=True)
    for r in range(g.n_rows):                       # the pair is the last kept entry's, or keeps everything
        cols = g.col_idx[g.row_ptr[r]: g.row_ptr[r + 1]]
        key, u = int(tk[r]) & M64, int(tu[r])
        if cols.size <= fanout:
            assert (key, u) == (M64, 0x7fffffff)
        else:
            kept = cols[okeep[g.row_ptr[r]: g.row_ptr[r + 1]] == 1]
            assert (key, u) == max((oracle.edge_key(77, r, int(c), 1), int(c)) for c in kept)


def _time_us(f):
    f()
    times = []
    for _ in range(3):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record(), f(), b.record()
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b) * 1e3)
    return min(times)


def test_cost_of_long_rows():
    """A long row is read a fixed number of times whatever the fanout (once per kept entry would be 100 times as much here), and
    long rows that follow each other in the list are not taken one after the other by one wavefront (16 times as much)."""
    import paper_2311_06837_amd as P
    ln, n_cols = 60000, 200000
    def mask(rows_of_it, fanout):
        lens = torch.tensor([ln] * rows_of_it + [5] * (400 - rows_of_it), device="cuda")
        rp = torch.zeros(401, dtype=torch.int32, device="cuda")
        rp[1:] = torch.cumsum(lens, 0)
        at = torch.arange(int(rp[-1]), device="cuda") - torch.repeat_interleave(rp[:-1], lens)
        G = P.Graph(rp, (at * 3).int(), n_cols=n_cols, sorted_columns=True)
        return _time_us(lambda: P.gnn_layer_edge_mask(G, None, 400, "fanout", 1, 5, fanout=fanout))
    one = mask(1, 10)
    assert mask(1, 100) < 6 * one and mask(1, 960) < 6 * one, "the cost grows with the fanout"
    assert mask(32, 10) < 4 * one, "consecutive long rows wait for each other"


def _mix64(x):
    with np.errstate(over="ignore"):
        x = x + np.uint64(0x9E3779B97F4A7C15)
        x = (x ^ (x >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        x = (x ^ (x >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        return x ^ (x >> np.uint64(31))


@pytest.mark.parametrize("fanout", [1, 15, 16, 31, 32, 33, 58, 59, 255, 256])
def test_fanouts_around_the_places_of_a_row(fanout):
    """Four rows of a wavefront that fit half of their places, or of which one does not (32); a quarter of a wavefront's registers
    (256); long rows whose list begins at nothing (58) or not."""
    short = [1, 16, 17, 31, 32, 32, 5, 0, 33, 2, 3, 4, 32, 31, 30, 34, 48, 63, 64, 1]
    _mask_case(_rows_of(short + [65, 128, 255, 256, 257, 258, 511, 1023, 1025, 2000, 9000] * 2, 30000, fanout + 1), None, "fanout", fanout, 2, 5)


@pytest.mark.parametrize("length", [40, 64, 65, 700, 1024, 1025, 3000])
def test_masks_when_the_upper_halves_of_two_keys_are_equal(length):
    """The selection compares upper halves of keys and falls back to whole pairs when the k-th is not alone with its half:
    rows built around two columns whose keys share the upper half, kept both, one of them, or neither.  Lengths on both
    sides of every class of rows."""
    n, layer, seed, v = 1_500_000, 1, 77, 5
    assert int(_mix64(_mix64(_mix64(np.uint64(seed + layer)) ^ np.uint64(v)) ^ np.uint64(123))) == oracle.edge_key(seed, v, 123, layer)
    keys = _mix64(_mix64(_mix64(np.uint64(seed + layer)) ^ np.uint64(v)) ^ np.arange(n, dtype=np.uint64))
    order = np.argsort(keys)
    half = keys[order] >> np.uint64(32)
    at = np.flatnonzero(half[1:] == half[:-1])
    assert at.size > 50                                        # about n^2 / 2^33 of them
    at = int(at[at > length][0])                               # the pair is order[at], order[at + 1]
    for k in (1, 2, 3, 10, 25):
        # the k-th smallest key is the first or the second of the pair, or lies before it
        for before in sorted({max(k - 1, 0), max(k - 2, 0), k}):
            if before + 2 > length:
                continue
            low = order[np.random.default_rng(before).choice(at, before, replace=False)]
            high = order[at + 2:][np.random.default_rng(k).choice(n - at - 2, length - before - 2, replace=False)]
            cols = np.sort(np.concatenate([low, order[at: at + 2], high])).astype(np.int32)
            row_ptr = np.zeros(n + 1, dtype=np.int32)
            row_ptr[v + 1:] = length
            _mask_case(gg.CSR(n, n, row_ptr, cols), np.array([v]), "fanout", k, layer, seed)


@pytest.mark.parametrize("sampler", [False, True])
def test_two_equal_upper_halves_cost_no_round_for_every_entry_kept(sampler):
    """One row of 1000 entries, fanout 600: with two equal halves among the smallest (0.5 ms, when the rounds went over all
    pairs) and without."""
    import paper_2311_06837_amd as P
    n, layer, seed, v, length, k = 1_500_000, 1, 77, 5, 1000, 600
    keys = _mix64(_mix64(_mix64(np.uint64(seed + layer)) ^ np.uint64(v)) ^ np.arange(n, dtype=np.uint64))
    order = np.argsort(keys)
    half = keys[order] >> np.uint64(32)
    at = np.flatnonzero(half[1:] == half[:-1])
    at = int(at[at > length][0])
    rng = np.random.default_rng(0)
    before = np.sort(rng.choice(at, k - 2, replace=False))
    after = at + 2 + rng.choice(n - at - 2, length - k, replace=False)
    us = []
    for pair in ([at, at + 1], [at, at + 2]):
        cols = np.unique(order[np.concatenate([before, pair, after])])
        cols = cols[cols != v].astype(np.int32)
        row_ptr = np.zeros(n + 1, np.int32)
        row_ptr[v + 1:] = cols.size
        G = P.Graph(dev(row_ptr), dev(cols), sorted_columns=True)
        rows, ws = dev(np.array([v], np.int32)), P.Workspace()
        bits = P.gnn_make_bitmap(rows, n)
        if sampler:
            call = lambda: P.gnn_sample_boundary(G, bits, rows, k, seed, ws=ws)
            got = call()[1]
            assert got.numel() == k
        else:
            call = lambda: P.gnn_layer_edge_mask(G, rows, 1, "fanout", layer, seed, fanout=k)
            got = dev(cols)[torch.from_numpy(_bits(call()[0], cols.size).astype(bool)).cuda()]
        want = cols[np.argsort(keys[cols])[:k]]
        assert np.array_equal(np.sort(got.cpu().numpy()), np.sort(want))
        times = []
        for _ in range(5):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(5):
                call()
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b) * 200)
        us.append(min(times))
    print(us, flush=True)
    assert us[0] < 1.3 * us[1]


def test_transposed_mask_rows_across_chunks():
    """A workgroup decides 4096 consecutive entries: rows that span several, runs of empty rows at the joints, a last chunk
    that ends inside a word."""
    import paper_2311_06837_amd as P
    n = 70000
    lengths = np.zeros(n, dtype=np.int64)
    lengths[[0, 1, 5, 6, 30000, 30001, n - 2]] = [4095, 1, 12289, 63, 64, 4096, 77]
    lengths[40000:40300] = np.random.default_rng(1).integers(0, 40, 300)
    rng = np.random.default_rng(2)
    cols = np.concatenate([np.sort(rng.choice(n, ln, replace=False)) for ln in lengths if ln] + [np.zeros(0)]).astype(np.int32)
    gt = gg.CSR(n, n, np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32), cols)
    assert gt.nnz % 32 not in (0, 1) and gt.nnz > 5 * 4096
    g = gg.transpose(gt)
    G, GT = P.Graph.from_numpy(g.row_ptr, g.col_idx), P.Graph.from_numpy(gt.row_ptr, gt.col_idx)
    for rule, kw in (("threshold", dict(threshold=oracle.keep_threshold(0.5))), ("fanout", dict(fanout=1))):
        keep, _, tk, tu = P.gnn_layer_edge_mask(G, None, n, rule, 3, 11, with_thresholds=True, **kw)
        kt = P.gnn_layer_edge_mask_transposed(GT, tk, tu, 3, 11)
        ok, _ = oracle.layer_edge_mask(g.row_ptr, g.col_idx, None, rule, 3, 11, **kw)
        assert np.array_equal(_bits(keep, g.nnz), ok), rule
        assert np.array_equal(_bits(kt, gt.nnz), oracle.transpose_mask(g.row_ptr, g.col_idx, ok, gt.row_ptr, gt.col_idx)), rule
        tail = int(kt.cpu().numpy().view(np.uint32)[-1]) >> (gt.nnz % 32)
        assert tail == 0, "bits past the last entry are set"


@pytest.mark.parametrize("run", [32700, 32800, 400_000])
def test_transposed_mask_across_long_runs_of_empty_rows(run):
    """Chunks whose entries lie on both sides of more empty rows than a workgroup walks (8 * 4096): in the middle of a chunk, at
    its first and at its last entry."""
    import paper_2311_06837_amd as P
    lengths = [0] * run + [4090, 5] + [0] * run + [1, 4096] + [0] * run + [4096, 3, 0, 0, 9] + [0] * run + [700] + [0] * run
    n, m = len(lengths), 6000
    rng = np.random.default_rng(run)
    rp = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    cols = np.concatenate([np.sort(rng.choice(m, ln, replace=False)) for ln in lengths if ln]).astype(np.int32)
    gt = gg.CSR(n, m, rp, cols)
    g = gg.transpose(gt)
    G = P.Graph.from_numpy(g.row_ptr, g.col_idx, n_cols=n)
    GT = P.Graph.from_numpy(gt.row_ptr, gt.col_idx, n_cols=m)
    keep, _, tk, tu = P.gnn_layer_edge_mask(G, None, m, "fanout", 2, 13, fanout=2, with_thresholds=True)
    kt = P.gnn_layer_edge_mask_transposed(GT, tk, tu, 2, 13)
    ok, _ = oracle.layer_edge_mask(g.row_ptr, g.col_idx, None, "fanout", 2, 13, fanout=2)
    assert np.array_equal(_bits(keep, g.nnz), ok)
    assert np.array_equal(_bits(kt, gt.nnz), oracle.transpose_mask(g.row_ptr, g.col_idx, ok, gt.row_ptr, gt.col_idx))


@pytest.mark.parametrize("n_cols,per_col", [(399_999, 4), (400_000, 4), (400_003, 5)])
def test_transposed_mask_of_many_columns(n_cols, per_col):
    """From 400 000 columns on an entry looks at the upper 16 bits of its column's key first.  Pairs that are an entry's own, one less or
    one more in key or id, with equal upper bits all of them, and the keys' extremes; with a workspace and without."""
    import ctypes as C
    import paper_2311_06837_amd as P
    from paper_2311_06837_amd import binding as B
    rng = np.random.default_rng(n_cols)
    n, nnz, layer, seed = 999, n_cols * per_col, 2, 12345
    cols = rng.permutation(np.arange(nnz, dtype=np.int64) % n_cols).astype(np.int32)
    at = np.sort(rng.integers(0, nnz + 1, n - 1))
    gt = gg.CSR(n, n_cols, np.concatenate([[0], at, [nnz]]).astype(np.int32), cols)
    u = np.repeat(np.arange(n, dtype=np.uint64), np.diff(gt.row_ptr))

    def mix(x):      # splitmix64's finaliser, as the header's key
        x = x + np.uint64(0x9E3779B97F4A7C15)
        x = (x ^ (x >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        x = (x ^ (x >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        return x ^ (x >> np.uint64(31))
    key = mix(mix(mix(np.full(1, seed + layer, dtype=np.uint64)) ^ cols.astype(np.uint64)) ^ u)
    own = np.zeros(n_cols, dtype=np.int64)
    own[cols] = np.arange(nnz)                                  # one entry of every column
    thr_k, thr_u = key[own].copy(), u[own].astype(np.int32)
    how = rng.integers(0, 8, n_cols)
    thr_u[how == 1] -= 1
    thr_u[how == 2] += 1
    thr_k[how == 3] -= np.uint64(1)
    thr_k[how == 4] += np.uint64(1)
    thr_k[how == 5] ^= np.uint64(1 << 47)                       # the upper bits stay
    thr_k[how == 6], thr_u[how == 6] = 0, -1
    thr_k[how == 7], thr_u[how == 7] = np.uint64(2 ** 64 - 1), 2 ** 31 - 1
    want = (key < thr_k[cols]) | ((key == thr_k[cols]) & (u.astype(np.int64) <= thr_u[cols]))
    GT = P.Graph.from_numpy(gt.row_ptr, gt.col_idx, n_cols=n_cols)
    tk, tu = dev(thr_k.view(np.int64)), dev(thr_u)
    need = C.c_size_t(1)
    args = (C.byref(GT.c), tk.data_ptr(), tu.data_ptr(), seed, layer)
    B._check(B.lib().gnn_layer_edge_mask_transposed_ws(*args, None, None, C.byref(need), None))
    assert (need.value > 0) == (n_cols >= 400_000)
    assert np.array_equal(_bits(P.gnn_layer_edge_mask_transposed(GT, tk, tu, layer, seed), nnz), want)
    plain = torch.empty((nnz + 31) // 32, dtype=torch.int32, device="cuda")
    B._check(B.lib().gnn_layer_edge_mask_transposed(*args, plain.data_ptr(), B._stream()))
    assert np.array_equal(_bits(plain, nnz), want)


def test_a_short_transposed_mask_asks_for_no_workspace(monkeypatch):
    """Below a million entries the answer is always none, and the question costs as much as a third of the call."""
    import paper_2311_06837_amd as P
    from paper_2311_06837_amd import binding as B
    g = gg.erdos_renyi(30_000, 20.0, 9)
    G = P.Graph.from_numpy(g.row_ptr, g.col_idx)
    _, _, tk, tu = P.gnn_layer_edge_mask(G, None, G.n_rows, "fanout", 1, 5, fanout=4, with_thresholds=True)
    want = P.gnn_layer_edge_mask_transposed(G, tk, tu, 1, 5)

    def refuse(*args):
        raise AssertionError("asked")
    monkeypatch.setattr(B.lib(), "gnn_layer_edge_mask_transposed_ws", refuse)
    assert torch.equal(P.gnn_layer_edge_mask_transposed(G, tk, tu, 1, 5), want)
    keep = P.gnn_layer_edge_mask(G, None, G.n_rows, "fanout", 1, 5, fanout=4)[0]
    assert torch.equal(P.gnn_transpose_edge_mask(G, G, keep), want)
    assert G.nnz < 1 << 20


def test_cost_of_empty_rows_in_the_transposed_mask():
    """Four million empty rows between two entries are not walked by the one workgroup that meets them (200 times the cost of
    the same rows behind the last entry)."""
    import paper_2311_06837_amd as P
    def mask(before, between, after):
        lens = torch.tensor([0] * before + [20] * 5000 + [0] * between + [20] * 5000 + [0] * after, device="cuda")
        rp = torch.zeros(lens.numel() + 1, dtype=torch.int32, device="cuda")
        rp[1:] = torch.cumsum(lens, 0)
        at = torch.arange(int(rp[-1]), device="cuda") % 20
        G = P.Graph(rp, at.int(), n_cols=20, sorted_columns=True)
        k, u = torch.zeros(20, dtype=torch.int64, device="cuda"), torch.zeros(20, dtype=torch.int32, device="cuda")
        return _time_us(lambda: P.gnn_layer_edge_mask_transposed(G, k, u, 1, 3))
    many = 4_000_000
    behind = mask(0, 0, many)
    assert mask(0, many, 0) < 12 * behind and mask(many, 0, 0) < 12 * behind


def test_transposed_mask():
    import paper_2311_06837_amd as P
    for g in (gg.random_directed(20000, 6.0, 4), gg.chung_lu(9000, 40.0, 2.1, 5)):
        gt = gg.transpose(g)
        G, keep, okeep = _mask_case(g, None, "threshold", oracle.keep_threshold(0.4), 2, 7)
        GT = P.Graph.from_numpy(gt.row_ptr, gt.col_idx)
        kt = P.gnn_transpose_edge_mask(G, GT, keep)
        torch.cuda.synchronize()
        want = oracle.transpose_mask(g.row_ptr, g.col_idx, okeep, gt.row_ptr, gt.col_idx)
        assert np.array_equal(_bits(kt, gt.nnz), want)
        # the same mask from the per-row threshold pairs, both rules, with only some rows listed
        rows = np.sort(np.random.default_rng(1).choice(g.n_rows, g.n_rows // 3, replace=False)).astype(np.int32)
        for rule, kw in (("threshold", dict(threshold=oracle.keep_threshold(0.4))), ("fanout", dict(fanout=3)), ("fanout", dict(fanout=0))):
            keep2, _, tk, tu = P.gnn_layer_edge_mask(G, dev(rows), len(rows), rule, 2, 7, with_thresholds=True, **kw)
            kt2 = P.gnn_layer_edge_mask_transposed(GT, tk, tu, 2, 7)
            torch.cuda.synchronize()
            ok2, _ = oracle.layer_edge_mask(g.row_ptr, g.col_idx, rows, rule, 2, 7, **kw)
            assert np.array_equal(_bits(keep2, g.nnz), ok2)
            assert np.array_equal(_bits(kt2, gt.nnz), oracle.transpose_mask(g.row_ptr, g.col_idx, ok2, gt.row_ptr, gt.col_idx)), rule


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("F,ld", [(64, 64), (128, 128), (256, 256), (602, 608), (100, 100), (7, 7)])
def test_aggregation_through_a_mask_forward_and_backward(dtype, F, ld):
    import paper_2311_06837_amd as P
    g = gg.chung_lu(8000, 60.0, 2.1, 21)                      # symmetric, a few rows above 1024 neighbours
    n = g.n_rows
    rng = np.random.default_rng(F)
    T = np.sort(rng.choice(n, 40, replace=False)).astype(np.int32)
    dist, ring, off = oracle.active_sets(g.row_ptr, g.col_idx, T, 2)
    rows = ring[: off[2]]                                      # R of a layer: targets and their neighbours
    print(f"masked aggregation: F={F} ld={ld} {dtype} rows={len(rows)}", flush=True)
    okeep, olen = oracle.layer_edge_mask(g.row_ptr, g.col_idx, rows, "fanout", 2, 3, fanout=6)
    rs = oracle.norm_scales("mean", olen)
    cs = (rng.random(n) + 0.5)
    X = as_stored(rng.standard_normal((n, F)), dtype)
    G = P.Graph.from_numpy(g.row_ptr, g.col_idx).with_edge_keep(_pack(okeep))
    Xd = padded(X, ld, dtype, fill=float("nan") if ld > F else 0.0)
    Yd = torch.full((n, ld), SENT, dtype=dtype, device="cuda")
    P.gnn_masked_spmm_fwd(G, dev(rows), len(rows), Xd, Yd, F, dev(rs.astype(np.float32)), dev(cs.astype(np.float32)), ws=P.Workspace())
    torch.cuda.synchronize()
    want = np.full((n, F), SENT)
    oracle.spmm_fwd_em(g.row_ptr, g.col_idx, okeep, rows, X, want, F, rs.astype(np.float32).astype(np.float64), cs.astype(np.float32).astype(np.float64))
    got = host64(Yd)
    check(got[rows, :F], want[rows], dtype, "forward")
    rest = np.setdiff1d(np.arange(n), rows)
    sent = host64(torch.tensor(SENT, dtype=dtype))
    assert (got[rest] == sent).all() and (got[:, F:] == sent).all()

    # backward: gather over the transposed graph (the graph is symmetric: same arrays) with the transposed mask and the
    # dist filter "v was a row of the forward call"
    kt = oracle.transpose_mask(g.row_ptr, g.col_idx, okeep, g.row_ptr, g.col_idx)
    GT = P.Graph.from_numpy(g.row_ptr, g.col_idx).with_edge_keep(_pack(kt))
    dY = as_stored(rng.standard_normal((n, F)), dtype)
    dYd = padded(dY, ld, dtype, fill=float("nan") if ld > F else 0.0)
    out_rows = ring[: off[3]]
    dXd = torch.full((n, ld), SENT, dtype=dtype, device="cuda")
    P.gnn_masked_spmm_bwd(GT, dev(out_rows), len(out_rows), dev(dist), 1, dYd, dXd, F, dev(rs.astype(np.float32)), dev(cs.astype(np.float32)),
                          accumulate=False)
    torch.cuda.synchronize()
    dX = np.zeros((n, F))
    oracle.spmm_bwd_em(g.row_ptr, g.col_idx, okeep, rows, dY, dX, F, rs.astype(np.float32).astype(np.float64), cs.astype(np.float32).astype(np.float64))
    got = host64(dXd)
    check(got[out_rows, :F], dX[out_rows], dtype, "backward")
    rest = np.setdiff1d(np.arange(n), out_rows)
    assert (got[rest] == sent).all() and (got[:, F:] == sent).all()


@pytest.mark.parametrize("kind,dtype,ls,dims", [
    ("sage", torch.float32, ("fanout", 4, 11), [32, 64, 48, 8]),
    ("gcn", torch.float32, ("threshold", oracle.keep_threshold(0.5), 12), [32, 64, 48, 8]),
    ("sage", torch.bfloat16, ("threshold", oracle.keep_threshold(0.7), 13), [32, 64, 48, 8]),
    ("sage", torch.float32, ("threshold", M64, 14), [32, 64, 48, 8]),
    # a first layer that narrows its input: the model multiplies by the weights first and aggregates the layer-1 mask
    # backward as well (its transposed mask is built too)
    ("sage", torch.float32, ("fanout", 4, 15), [64, 32, 48, 8]),
    ("sage", torch.float32, ("threshold", oracle.keep_threshold(0.5), 16), [64, 32, 48, 8])])
def test_training_step_with_per_layer_masks(kind, dtype, ls, dims):
    import paper_2311_06837_amd as P
    w = gg.make_workload("cfg0", scale=0.5)
    part = w.partition
    print(f"model with layer sampling {ls[0]}: n={part.graph.n_rows} nnz={part.graph.nnz} {kind} {dtype}", flush=True)
    L = len(dims) - 1
    g = part.graph if kind == "sage" else part.graph
    T = part.targets
    # three layers over a 2-hop partition: the outermost active set simply repeats
    params = gg.layer_weights(dims, kind == "sage", 5)
    n = g.n_rows
    H0 = as_stored(gg.features(n, dims[0], 5), dtype)
    y = gg.labels(len(T), dims[-1], 5)
    gdeg = part.global_degree if kind == "gcn" else None
    om = oracle.Model(g.row_ptr, g.col_idx, T, kind, params, gdeg, bf16=dtype == torch.bfloat16, layer_sampling=ls)
    loss_o = om.forward(H0, y)
    grads_o = om.backward()
    G = P.Graph.from_numpy(g.row_ptr, g.col_idx)
    m = P.MaskedGNN(G, G, dev(T), kind, [{k: dev(v) for k, v in p.items()} for p in params], dtype=dtype,
                    global_degree=dev(gdeg) if gdeg is not None else None, layer_sampling=ls,
                    transform_first=True)      # every narrowing layer in the exchanged order
    assert m.tf_layers == {l for l in range(1, L + 1) if dims[l - 1] > dims[l]}   # (asked for below)
    m.set_input(padded(H0, P.row_stride(dims[0], dtype), dtype))
    loss = m.step(dev(y))
    torch.cuda.synchronize()
    for l in range(1, L + 1):
        assert np.array_equal(_bits(m.g_l[l].edge_keep, g.nnz), om.keep[l]), f"mask of layer {l}"
    tol = TOL[dtype]
    assert abs(loss.item() - loss_o) <= tol * L * abs(loss_o), (loss.item(), loss_o)
    backward_at_the_oracles_point(m, om, dims, dtype, dev(y))     # same ReLU decisions on both sides, then element by element
    for l in range(L):
        for k, want in grads_o[l].items():
            check(host64(m.grads[l][k]), want, dtype, f"layer {l + 1} {k}", calls=L - l)
    if ls[1] == M64:       # everything kept: the plain model
        plain = oracle.Model(g.row_ptr, g.col_idx, T, kind, params, gdeg, bf16=dtype == torch.bfloat16)
        assert plain.forward(H0, y) == loss_o
