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
