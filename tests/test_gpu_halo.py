"""GPU parity of halo partitions: bit-exact construction, and a train step over the owned
nodes of a k-hop halo partition against the oracle (which pins it to the whole-graph step)."""
import numpy as np
import pytest
import torch

import synth
from oracle import graph as ograph
from oracle import step as ostep
from tests._cases import TOL_FP32, assert_step_grads_close

pytestmark = pytest.mark.gpu
DEV = "cuda"
KEYS = ("l2g", "rowptr", "col", "colptr", "row", "d_local_in", "d_local_out", "d_global_in")


@pytest.fixture(scope="module")
def g():
    import paper_2602_01872_amd as lib
    lib.load()
    return lib


@pytest.mark.parametrize("kind,N,E,K,hops", [("uniform", 5000, 30000, 4, 1), ("uniform", 5000, 30000, 4, 2),
                                              ("rmat", 1 << 13, 100000, 8, 1), ("rmat", 1 << 13, 100000, 8, 3),
                                              ("uniform", 400, 0, 2, 1),
                                              # two ranges of local ids to count in-degrees by; a last tile of edges that is not whole
                                              ("uniform", 30000, 200001, 3, 1), ("uniform", 30000, 60000, 2, 2)])
def test_partition_halo_bit_exact(g, kind, N, E, K, hops):
    print(f"[case] halo partition {kind} N={N} E={E} K={K} hops={hops}", flush=True)
    if E == 0:
        s = d = torch.zeros(0, dtype=torch.int64)
    elif kind == "uniform":
        s, d = synth.uniform_graph(N, E, seed=61)
    else:
        s, d = synth.rmat_graph(13, E, seed=61)
    for p in (0, K - 1):
        part = g.grp_partition_halo(s.to(DEV), d.to(DEV), N, K, 7, p, hops)
        want = ograph.partition_halo(s.numpy(), d.numpy(), N, K, 7, p, hops)
        assert part.n == want["n"] and part.nnz == want["nnz"]
        for k in KEYS:
            assert np.array_equal(part.array(k), want[k]), k
        assert np.array_equal(part.base_mask(), want["owned_mask"])
        part.destroy()
    with pytest.raises(g.GrappaError):
        g.grp_partition_halo(s.to(DEV), d.to(DEV), N, K, 7, 0, 0)
    if E:
        bad = d.clone(); bad[5] = -1
        with pytest.raises(g.GrappaError) as ei:
            g.grp_partition_halo(s.to(DEV), bad.to(DEV), N, K, 7, 0, 1)
        assert ei.value.status == g.ERANGE


def assert_equal_to_oracle(g, s, d, N, K, p, hops, on=None):
    want = ograph.partition_halo(s.numpy(), d.numpy(), N, K, 7, p, hops)
    part = g.grp_partition_halo(*(on or (s.to(DEV), d.to(DEV))), N, K, 7, p, hops)
    assert part.n == want["n"] and part.nnz == want["nnz"]
    for k in KEYS:
        assert np.array_equal(part.array(k), want[k]), k
    assert np.array_equal(part.base_mask(), want["owned_mask"])
    part.destroy()
    return want


def one_node_graph(E, K, at_hop):
    """E edges from everywhere into one node of partition 0 (at_hop 0), or into the source of an edge that ends in one."""
    N = 20_000
    own = ograph.owner(N, K, 7) == 0
    s, d = synth.uniform_graph(N, E, seed=66)
    d[:] = int(np.flatnonzero(own if at_hop == 0 else ~own)[3])
    if at_hop:
        s[E // 2], d[E // 2] = int(d[0]), int(np.flatnonzero(own)[5])
    return N, s, d


@pytest.mark.parametrize("at_hop,hops", [(0, 1), (1, 2), (1, 1)])
def test_halo_of_one_busy_node(g, at_hop, hops):
    """All edges end in one node.  If it is owned, one hop keeps more of them than twice a partition's share and 2^20: their keys are written once
    more, to a buffer of their number."""
    E, K = 3_000_001, 8
    N, s, d = one_node_graph(E, K, at_hop)
    print(f"[case] halo overflow E={E} at_hop={at_hop} hops={hops}", flush=True)
    want = assert_equal_to_oracle(g, s, d, N, K, 0, hops)
    assert want["nnz"] == (E if at_hop < hops else 1) and E > 2 * (E // K) + (1 << 20)


@pytest.mark.parametrize("hops", [1, 2])
def test_halo_of_more_than_2_to_22_members(g, hops):
    N, E, K = (1 << 23) + (1 << 17), 200_001, 2
    print(f"[case] halo N={N} E={E} hops={hops}", flush=True)
    s, d = synth.uniform_graph(N, E, seed=67)
    assert assert_equal_to_oracle(g, s, d, N, K, 1, hops)["n"] > 1 << 22


def test_halo_edges_that_are_not_aligned(g):
    """Edge arrays that begin 8 bytes past a 16-byte boundary are read one id at a time."""
    N, E, K = 30_000, 200_001, 3
    s, d = synth.uniform_graph(N, E, seed=68)
    on = [torch.empty(E + 1, dtype=torch.int64, device=DEV)[1:].copy_(t) for t in (s, d)]
    assert all(t.data_ptr() % 16 == 8 for t in on)
    for hops in (1, 2):
        print(f"[case] halo unaligned hops={hops}", flush=True)
        assert_equal_to_oracle(g, s, d, N, K, 0, hops, on)


def test_halo_without_room_for_the_scratch(g):
    """Where there is no room for the keys and ids of one pass (720 MB here; the partition itself takes 2), the build counts first."""
    N, E, K = 20_000, 60_000_000, 2
    own = ograph.owner(N, K, 7) == 0
    s, d = torch.zeros(E, dtype=torch.int64, device=DEV), torch.full((E,), int(np.flatnonzero(~own)[3]), dtype=torch.int64, device=DEV)
    s[:50_000], d[:50_000] = (t.to(DEV) for t in synth.uniform_graph(N, 50_000, seed=69))
    first = g.grp_partition_halo(s, d, N, K, 7, 0, 1)      # (first use: code objects and the like)
    want = {k: first.array(k) for k in KEYS}
    first.destroy()
    g.grp_release_memory()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    # All memory in pieces of 150 MB (more of them than the runtime says that there are), but for two.
    piece, rest = 150 << 20, [torch.empty(torch.cuda.mem_get_info()[0] - (1 << 30), dtype=torch.uint8, device=DEV)]
    try:
        while len(rest) < 200:
            try:
                rest.append(torch.empty(piece, dtype=torch.uint8, device=DEV))
            except torch.cuda.OutOfMemoryError:
                break
        print(f"[case] halo build with two of {len(rest) - 1} pieces left", flush=True)
        assert 2 < len(rest) < 200
        del rest[-2:]
        torch.cuda.empty_cache()
        part = g.grp_partition_halo(s, d, N, K, 7, 0, 1)
    finally:
        del rest
        torch.cuda.empty_cache()
    for k in KEYS:
        assert np.array_equal(part.array(k), want[k]), k
    assert part.nnz == len(want["col"]) < 1 << 17
    part.destroy()


@pytest.mark.parametrize("value", [-1, -2, 5000, -(1 << 40)])
@pytest.mark.parametrize("end", ["src", "dst"])
def test_halo_ids_out_of_range(g, end, value):
    """One id outside [0, N), at either end of an edge, in a whole tile of edges, in the tail and last of all: refused, whatever its value."""
    N, E, K = 5000, 30001, 4
    s, d = synth.uniform_graph(N, E, seed=61)
    for at in (5, E - 40, E - 1):
        bad = {"src": s.clone(), "dst": d.clone()}
        bad[end][at] = value
        for hops in (1, 2):
            print(f"[case] halo bad {end} {value} at {at} hops={hops}", flush=True)
            with pytest.raises(g.GrappaError) as ei:
                g.grp_partition_halo(bad["src"].to(DEV), bad["dst"].to(DEV), N, K, 7, 0, hops)
            assert ei.value.status == g.ERANGE


def test_halo_of_no_nodes(g):
    """Without nodes every edge's ends are out of range."""
    none, some = torch.zeros(0, dtype=torch.int64, device=DEV), torch.zeros(3, dtype=torch.int64, device=DEV)
    part = g.grp_partition_halo(none, none, 0, 2, 7, 0, 1)
    assert part.n == part.nnz == 0
    part.destroy()
    with pytest.raises(g.GrappaError) as ei:
        g.grp_partition_halo(some, some, 0, 2, 7, 0, 1)
    assert ei.value.status == g.ERANGE


@pytest.mark.parametrize("arch,dims", [("sage", [12, 16, 5]), ("gat", [12, 16, 5])])
def test_train_step_on_a_k_hop_halo_partition(g, arch, dims):
    print(f"[case] halo train step {arch} {dims}", flush=True)
    N, E, K = 6000, 36000, 4
    s, d = synth.uniform_graph(N, E, seed=62)
    hops = len(dims) - 1
    part = g.grp_partition_halo(s.to(DEV), d.to(DEV), N, K, 3, 2, hops)
    op = ograph.partition_halo(s.numpy(), d.numpy(), N, K, 3, 2, hops)
    l2g = torch.from_numpy(op["l2g"])
    x = synth.normal_matrix(N, dims[0], 63)[l2g].contiguous()
    y = synth.labels(N, dims[-1], 64)[l2g].contiguous()
    theta = synth.model_weights(arch, dims, 65)
    model = g.model_desc(g.ARCH_SAGE_MEAN if arch == "sage" else g.ARCH_GAT, dims)
    opts = g.step_opts(estimator=g.EST_SHRINKAGE)
    P = g.grp_param_count(model)
    ws = torch.empty(g.grp_step_workspace_bytes(part, model, opts), dtype=torch.uint8, device=DEV)
    grad = torch.full((P,), float("nan"), device=DEV)
    stats = g.new_stats(1)
    mask = torch.from_numpy(part.base_mask()).to(DEV)
    g.grp_train_step(part, model, opts, x.to(DEV), y.to(DEV), mask, theta.to(DEV), ws, grad, stats)
    torch.cuda.synchronize()

    def oracle_fn(relu_flip=None, near_kink=None):
        return ostep.train_step(op, arch, dims, theta.double().numpy(), x.double().numpy(), y.numpy(), op["owned_mask"],
                                estimator=3, relu_flip=relu_flip, near_kink=near_kink)
    og, ost = assert_step_grads_close(grad.cpu().numpy(), oracle_fn, arch, dims, TOL_FP32)
    st = g.read_stats(stats)[0]
    assert int(st["S"]) == ost["S"] == int(op["owned_mask"].sum())
    assert float(st["R"]) == 0.0                      # every owned node sees its whole in-neighbourhood
    # and the oracle ties this to the whole graph restricted to the owned nodes
    whole = ograph.partition(s.numpy(), d.numpy(), N, 1, 0, 0)
    own = (ograph.owner(N, K, 3) == 2).astype(np.uint8)
    xg = synth.normal_matrix(N, dims[0], 63).double().numpy()
    yg = synth.labels(N, dims[-1], 64).numpy()
    gw, _ = ostep.train_step(whole, arch, dims, theta.double().numpy(), xg, yg, own)
    np.testing.assert_allclose(og, gw, rtol=1e-9, atol=1e-12)
    part.destroy()
