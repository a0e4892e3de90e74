"""Rows that end at the last position an int32 can name: a graph of 2^31 - 1 entries, the most the interface accepts.  Every call
must give what it gives for the same rows in a small graph; a position past a row's end must not wrap around to a negative one."""
import ctypes as C

import numpy as np
import pytest
import torch

from gpu_util import dev

pytestmark = pytest.mark.gpu

NNZ = 2 ** 31 - 1
N = 9000                # vertex N - 1 has the row in question; vertex 0 holds all other entries and is never looked at


@pytest.fixture(scope="module")
def columns():
    c = torch.zeros(NNZ, dtype=torch.int32, device="cuda")
    yield c
    del c
    torch.cuda.empty_cache()


def _both(columns, length):
    """The graph of NNZ entries whose last row has `length` of them, and the same row in a small graph."""
    import paper_2311_06837_amd as P
    row = np.sort(np.random.default_rng(length).choice(np.arange(1, N - 1), length, replace=False)).astype(np.int32)
    columns[NNZ - length:] = dev(row)
    out = []
    for cols, first in ((columns, NNZ - length), (dev(row), 0)):
        rp = torch.full((N + 1,), first, dtype=torch.int32, device="cuda")
        rp[0], rp[N] = 0, first + length
        out.append(P.Graph(rp, cols, sorted_columns=True))
    return out, row


def _bits_at(words, lo, hi):
    p = torch.arange(lo, hi, device="cuda")
    return ((words[p // 32] >> (p % 32)) & 1).cpu().numpy()


@pytest.mark.parametrize("length", [1, 60, 70, 1000, 1030, 2500, 7000])
def test_last_row_of_a_graph_of_as_many_entries_as_fit(columns, length):
    import paper_2311_06837_amd as P
    print(f"index limit: last row of {length}", flush=True)
    graphs, row = _both(columns, length)
    T = dev(np.array([N - 1], dtype=np.int32))
    X = torch.randn(N, 64, generator=torch.Generator(device="cuda").manual_seed(1), device="cuda")
    W = torch.randn(64, 32, generator=torch.Generator(device="cuda").manual_seed(2), device="cuda")
    keep_some = (torch.rand(N, generator=torch.Generator(device="cuda").manual_seed(3), device="cuda") < 0.5).int() - 1   # 0 or -1
    results = []
    for g in graphs:
        r = {}
        first, end = g.nnz - length, g.nnz
        dist, ring, off, hop = P.gnn_build_active_sets(g, T, 1)
        r["dist"], r["ring"], r["hop"] = dist, ring[: int(hop[-1])], off
        # every vertex that is not reached looks for the frontier through its row of the "transposed" graph: its last row too
        far, _, _, _ = P.gnn_build_active_sets(g, dev(row[:1]), 1, gt=g)
        r["far"] = far
        for rule in ("hash",):
            for fanout in (1, 40, 980):
                d, _, _, _ = P.gnn_eas_traverse(g, T, 1, fanout, rule, 5)
                r[f"eas {rule} {fanout}"] = d
        local, new_id = P.gnn_extract_partition(g, ring, int(hop[-1]), dist, 1)
        r["local rows"], r["local columns"], r["new_id"] = local.row_ptr, local.col_idx, new_id
        bits = P.gnn_make_bitmap(dev(np.concatenate([[N - 1], row[::3]]).astype(np.int32)), N)
        for fanout in (3, 200):
            rp, ci = P.gnn_sample_boundary(g, bits, T, fanout, 11)
            r[f"sampled {fanout}"], r[f"sampled columns {fanout}"] = rp, ci
        for rule, how in (("fanout", dict(fanout=7)), ("fanout", dict(fanout=300)), ("threshold", dict(threshold=1 << 62))):
            keep, kept_len, tk, tu = P.gnn_layer_edge_mask(g, T, 1, rule, 1, 9, with_thresholds=True, **how)
            name = f"mask {rule} {how}"
            r[name], r[name + " kept"] = torch.from_numpy(_bits_at(keep, first, end)), kept_len
            r[name + " thresholds"] = torch.cat([tk, tu.long()])
            if how == dict(fanout=7):
                Y = torch.zeros(N, 64, device="cuda")
                P.gnn_masked_spmm_fwd(g.with_edge_keep(keep), T, 1, X, Y, 64)
                r["masked aggregation"] = Y
        for F in (16, 64):
            Y = torch.zeros(N, F, device="cuda")
            P.gnn_masked_spmm_fwd(g, T, 1, X[:, :F].contiguous(), Y, F)
            r[f"aggregation {F}"] = Y
        Y = torch.zeros(N, 64, device="cuda")
        P.gnn_masked_spmm_bwd(g, T, 1, keep_some, 0, X, Y, 64)
        r["filtered aggregation"] = Y
        H = torch.zeros(N, 32, device="cuda")
        P.gnn_fused_layer_fwd(g, T, 1, X, 64, None, None, W, None, None, H, relu=False)
        r["fused layer"] = H
        torch.cuda.synchronize()
        results.append(r)
    for k, want in results[1].items():
        assert torch.equal(results[0][k], want), k
    want = X[torch.from_numpy(row).cuda().long()].double().sum(0)
    assert float((results[0]["aggregation 64"][N - 1].double() - want).norm() / want.norm()) < 1e-5
