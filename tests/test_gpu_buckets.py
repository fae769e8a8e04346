"""The builders' sort by buckets of rows: every array of the handle equals the oracle's, and the lists of long rows serve the
aggregation (whole numbers, so that sums are exact), at the edges of its tiles, buckets and counting jobs."""
import numpy as np
import pytest
import torch

from oracle import graph as ograph

pytestmark = pytest.mark.gpu
DEV = "cuda"
KEYS = ("l2g", "rowptr", "col", "colptr", "row", "d_local_in", "d_local_out", "d_global_in")


def _edges(kind, n, E, rng):
    s, d = rng.integers(0, n, E), rng.integers(0, n, E)
    if kind == "hub":                       # one row and one column of more keys than a workgroup sorts, over several ranges of ids
        d[: E // 2] = n // 3
        s[E // 2: E - E // 10] = n - 1
    elif kind == "same":                    # one pair, over and over
        s[:], d[:] = n - 1, 0
    elif kind == "crowded":                 # consecutive rows that fill a bucket several times over, none of them alone
        d[: E - E // 8] = n // 2 + rng.integers(0, 8, E - E // 8)
    elif kind == "near":                    # neighbours with close ids: many keys of a row in one range
        s = np.clip(d + rng.integers(-40, 40, E), 0, n - 1)
    elif kind == "near hub":                # the same, of a hub
        d[: E // 2], s[: E // 2] = n // 2, n // 3 + rng.integers(0, 9000, E // 2)
    elif kind == "last":                    # everything in the last row's bucket
        d[:] = n - 1 - rng.integers(0, 3, E) % n
    return s.astype(np.int64), d.astype(np.int64)


@pytest.mark.parametrize("kind,n,E", [
    ("uniform", 1, 1), ("uniform", 1, 9000), ("uniform", 2, 4097), ("uniform", 63, 128), ("uniform", 2049, 8192),
    ("uniform", 5000, 60001), ("hub", 40001, 60000), ("hub", 16385, 8193 * 2), ("same", 3, 20000), ("crowded", 2000, 27000),
    ("near", 3001, 400000), ("near hub", 65537, 150000), ("last", 70000, 300000), ("uniform", 1 << 22, 5000), ("uniform", (1 << 22) + 1, 5000), ("hub", 300000, 9000000),
])
def test_local_edges_bit_exact(kind, n, E):
    import paper_2602_01872_amd as g
    print(f"[case] buckets {kind} n={n} E={E}", flush=True)
    s, d = _edges(kind, n, E, np.random.default_rng(n + E))
    want = ograph.local_graph_from_edges(s, d, n)
    part = g.grp_partition_from_local_coo(torch.from_numpy(s).to(DEV), torch.from_numpy(d).to(DEV), n)
    assert part.nnz == E
    for k in KEYS:
        assert np.array_equal(part.array(k), want[k]), k
    if n > 1 << 20:
        return
    x = torch.arange(4 * n, device=DEV).remainder_(7).float().view(n, 4)
    sd, dd = torch.from_numpy(s).to(DEV), torch.from_numpy(d).to(DEV)
    for transposed, (a, b) in ((False, (sd, dd)), (True, (dd, sd))):
        y = torch.empty(n, 4, device=DEV)
        g.grp_spmm(part, transposed, g.SCALE_NONE, False, 4, x, 4, g.DTYPE_FP32, y, 4)
        assert torch.equal(y, torch.zeros(n, 4, device=DEV).index_add_(0, b, x[a])), transposed


@pytest.mark.parametrize("N,K", [(1, 1), (31, 2), (64, 3), (70001, 1), (70001, 6), (70001, 7), (70000, 48), (70000, 1 << 20), (70000, (1 << 31) - 1)])
def test_hash_split_bit_exact(N, K):
    import paper_2602_01872_amd as g
    rng = np.random.default_rng(N + K)
    s, d = rng.integers(0, N, 200001), rng.integers(0, N, 200001)
    owner = torch.empty(N, dtype=torch.int32, device=DEV)
    g.grp_node_owners(N, K, 5, owner)
    for p in sorted({0, K - 1, int(owner[N // 2])}):
        print(f"[case] hash N={N} K={K} part {p}", flush=True)
        want = ograph.partition(s, d, N, K, 5, p)
        part = g.grp_partition(torch.from_numpy(s).to(DEV), torch.from_numpy(d).to(DEV), N, K, 5, p)
        assert part.n == want["n"]
        for k in KEYS:
            assert np.array_equal(part.array(k), want[k]), k
