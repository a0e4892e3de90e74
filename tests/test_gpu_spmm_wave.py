"""The aggregation's kernel for short rows of large graphs (a wavefront walks its rows as one stream), against plain torch sums
in 64 bits: rows without entries, rows that fill whole batches of 64, long rows, row lists, a source prefix, widths that leave
lanes and parts of lanes idle, offsets beyond 32 bits."""
import numpy as np
import pytest
import torch

from test_gpu_spmm_split import _want

pytestmark = pytest.mark.gpu


def _graph(n, seed):
    rng = np.random.default_rng(seed)
    lens = rng.poisson(4.2, n)
    lens[rng.integers(0, n, 200)] = 64
    lens[rng.integers(0, n, 200)] = rng.integers(60, 70, 200)
    lens[rng.integers(0, n, 60)] = rng.integers(250, 1400, 60)
    lens[1000:1300] = 0
    lens[5] = 30_000
    lens[n - 1] = 257
    rows = np.repeat(np.arange(n, dtype=np.int64), lens)
    keys = np.unique(rows * n + rng.integers(0, n, len(rows)))
    row_ptr = np.zeros(n + 1, np.int64)
    row_ptr[1:] = np.cumsum(np.bincount(keys // n, minlength=n))
    return row_ptr.astype(np.int32), (keys % n).astype(np.int32)


@pytest.mark.parametrize("dtype,F,ld", [(torch.float32, 33, 36), (torch.float32, 64, 64), (torch.float32, 65, 68), (torch.float32, 128, 128),
                                        (torch.bfloat16, 65, 72), (torch.bfloat16, 128, 128), (torch.bfloat16, 130, 136), (torch.bfloat16, 256, 256),
                                        (torch.float32, 64, 7936)])
@pytest.mark.parametrize("form", ["scaled", "prefix", "list"])
def test_short_rows_of_a_large_graph(dtype, F, ld, form):
    import paper_2311_06837_amd as P
    if ld > 4096 and form == "list":
        pytest.skip("one of the 64-bit forms is enough")
    n = 140_003
    row_ptr, col = _graph(n, F)
    ci = torch.from_numpy(col).cuda()
    G = P.Graph(torch.from_numpy(row_ptr).cuda(), ci, sorted_columns=True)
    gen = torch.Generator(device="cuda").manual_seed(F)
    X = torch.full((n, ld), float("nan"), dtype=dtype, device="cuda")
    X[:, :F] = torch.randn(n, F, generator=gen, device="cuda").to(dtype)
    rs, cs = (torch.rand(n, generator=gen, device="cuda") + 0.5 for _ in range(2))
    if form == "prefix":
        cs = None
    Y = torch.full((n, F + (-F) % 8), 12345.0, dtype=dtype, device="cuda")
    n_active, limit, rows = n, n, None
    if form == "prefix":
        limit = int(n * 0.7)
        P.gnn_masked_spmm_bwd(G, None, n, None, 0, X, Y, F, cs, rs, accumulate=False, src_prefix=limit)
    else:
        if form == "list":
            rows = torch.randperm(n, generator=gen, device="cuda")[:120_001].int()
            n_active = rows.numel()
        P.gnn_masked_spmm_fwd(G, rows, n_active, X, Y, F, rs, cs)
    want, size, lens = _want(row_ptr, ci, n, X[:, :F], rs, cs, limit)
    tol = (lens + 8) * 2.0 ** -24 * size + (2.0 ** -8 * want.abs() if dtype == torch.bfloat16 else 0.0) + 1e-30
    got = Y[:, :F].double()
    if rows is not None:
        listed = torch.zeros(n, dtype=torch.bool, device="cuda")
        listed[rows.long()] = True
        assert (got[~listed] == torch.tensor(12345.0, dtype=dtype).double()).all(), "rows outside the list were written"
        got, want, tol = got[listed], want[listed], tol[listed]
    worst = ((got - want).abs() / tol).max().item()
    assert worst <= 1.0, worst
    assert (Y[:, F:] == torch.tensor(12345.0, dtype=dtype)).all(), "pad columns were written"
