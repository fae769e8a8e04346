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
    ("uniform", 1 << 22, 9_000_000),       # as many buckets as there may be, keys of 32 bits, the longest tiles of the scatter
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


@pytest.mark.parametrize("inside", [False, True])            # every edge within the part: more keys than one pass has room for
def test_hash_split_of_many_nodes_reads_the_edges_once(inside):
    """Parts of more than 2^22 nodes count their in-degrees another way, in the pass that writes the keys all the same."""
    import paper_2602_01872_amd as g
    N, K, E = 9_000_000, 2, 3_000_001
    print(f"[case] hash N={N} K={K} inside={inside}", flush=True)
    rng = np.random.default_rng(8)
    s, d = rng.integers(0, N, E), rng.integers(0, N, E)
    d[: E // 3] = 77                                        # a hub
    if inside:
        owner = torch.empty(N, dtype=torch.int32, device=DEV)
        g.grp_node_owners(N, K, 5, owner)
        own = torch.nonzero(owner == 1).flatten().cpu().numpy()
        assert len(own) > 1 << 22
        s, d = own[s % len(own)], own[d % len(own)]
    want = ograph.partition(s, d, N, K, 5, 1)
    g.grp_profile_enable(1)
    try:
        part = g.grp_partition(torch.from_numpy(s).to(DEV), torch.from_numpy(d).to(DEV), N, K, 5, 1)
        torch.cuda.synchronize()
        passes = [k for k in g.grp_profile_report() if k.startswith("partition_edge")]
    finally:
        g.grp_profile_enable(0)
    assert passes == ["partition_edge_scan_keys"] + ["partition_edge_keys"] * inside
    for k in KEYS:
        assert np.array_equal(part.array(k), want[k]), k


def _degrees(kind):
    W, C = 4096, 8192                       # keys by which a crowded bucket's rows are dealt to jobs; keys a workgroup sorts
    return {"edges of a job": [W - 1, 1, W, 0, W + 1, 3, C - 1, C, 0, C + 1, 2, W, W, W],
            "hub first and last": [C + 1, 5, 5, 0, 3 * C],
            "one after another": [W] * 9 + [W + 1] * 5,
            "a hub of one sort": [C + 1],
            "long hub": [(1 << 18) + 1, 7, 1 << 18],
            "few ranges": [C - 1, 2, C - 9], "few ranges, a hub": [7, 2 * C - 9], "jobs at once": [W, W, W, W, 1],
            "too long for a workgroup": [(1 << 20) + 1, 40],
            "too much for the hubs' jobs": [1_000_000, 1_000_000, 1_000_000, 40]}[kind]


@pytest.mark.parametrize("spread", [1, 300])                # rows beside each other, in a bucket each
@pytest.mark.parametrize("kind", ["edges of a job", "hub first and last", "one after another", "a hub of one sort", "long hub", "few ranges", "few ranges, a hub", "jobs at once",
                                  "too long for a workgroup", "too much for the hubs' jobs"])
def test_crowded_buckets_bit_exact(kind, spread):
    import paper_2602_01872_amd as g
    deg = _degrees(kind)
    n, E = 70_000, sum(deg) + 4000
    print(f"[case] crowded buckets {kind} spread={spread} E={E}", flush=True)
    rng = np.random.default_rng(E)
    rows = 100 + spread * np.arange(len(deg))
    a = rng.permutation(np.concatenate([np.repeat(rows, deg), rng.integers(0, n, 4000)]))
    b = np.where(rng.random(E) < 0.1, rng.integers(5, 12, E), rng.integers(0, n, E))      # (some ids of a row many times over)
    for s, d in ((a, b), (b, a)):
        want = ograph.local_graph_from_edges(s, d, n)
        part = g.grp_partition_from_local_coo(torch.from_numpy(s).to(DEV), torch.from_numpy(d).to(DEV), n)
        for k in KEYS:
            assert np.array_equal(part.array(k), want[k]), k
        x = torch.arange(4 * n, device=DEV).remainder_(3).float().view(n, 4)
        sd, dd = torch.from_numpy(s).to(DEV), torch.from_numpy(d).to(DEV)
        for transposed, (u, v) in ((False, (sd, dd)), (True, (dd, sd))):       # (sums below 2^24: exact)
            y = torch.empty(n, 4, device=DEV)
            g.grp_spmm(part, transposed, g.SCALE_NONE, False, 4, x, 4, g.DTYPE_FP32, y, 4)
            assert torch.equal(y, torch.zeros(n, 4, device=DEV).index_add_(0, v, x[u])), transposed


def test_heavy_rows_beside_each_other_cost_no_more_than_scattered_ones():
    """150 popular nodes, numbered first: once read again for every one of them, 85 ms against 0.34 scattered."""
    import paper_2602_01872_amd as g
    n, E, popular = 300_000, 3_000_000, 150
    gen = torch.Generator(device=DEV).manual_seed(1)
    s = popular + torch.randint(n - popular, (E,), generator=gen, device=DEV)
    d = torch.randint(popular, (E,), generator=gen, device=DEV)
    perm = torch.randperm(n, generator=gen, device=DEV)

    def best(s, d):
        times = []
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            g.grp_partition_from_local_coo(s, d, n).destroy()
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b))
        return min(times)
    keep = g.grp_partition_from_local_coo(s[:4], d[:4], n)
    assert best(s, d) < 20 * best(perm[s], perm[d])
    keep.destroy()
