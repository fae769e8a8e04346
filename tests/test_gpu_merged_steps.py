"""Steps whose launches are merged give the bits that the same steps give one after another: partitions of very different sizes (other tiles, more
or fewer launches: long rows, slices of the sums), more steps than one launch takes, steps with launches that are not merged, steps that are
made one by one.  What is merged is seen by the number of launches."""
import ctypes

import pytest
import torch

import synth
from tests._cases import make_inputs

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _graph(n, E, seed):
    s, d = synth.rmat_graph(max(2, (n - 1).bit_length()), E, seed=seed, n_nodes=n)
    return s.to(DEV), d.to(DEV)


@pytest.mark.parametrize("arch,dims,sizes,dropout", [
    ("gcn", [64, 64, 8], [(2500, 6000), (2400, 40000), (1, 0), (9000, 20000)], 0.0),
    ("gcn", [17, 33, 5], [(300, 900)] * 11, 0.25),                 # two launches of eight and three; scaled weights
    ("gcn_res", [32, 32, 32, 6], [(700, 5000), (4100, 9000)], 0.5),
    ("sage", [30, 100, 70, 200], [(5000, 60000), (64, 100), (40000, 90000)], 0.5),      # more classes than a row's lanes hold
    ("sage", [24, 16, 16, 16, 16, 8], [(800, 4000)] * 3, 0.5),     # more weights than a merged launch's arguments hold
    ("sage", [30, 3, 2], [(800, 4000)] * 3, 0.0),                  # rows narrower than a vector
    ("gat", [12, 16, 4], [(500, 3000), (600, 3000)], 0.0),         # (one by one)
])
def test_full_graph_steps(arch, dims, sizes, dropout):
    import paper_2602_01872_amd as g
    print(f"[case] merged {arch} {dims} {sizes}", flush=True)
    code = {"sage": g.ARCH_SAGE_MEAN, "gcn": g.ARCH_GCN, "gcn_res": g.ARCH_GCN_RESIDUAL, "gat": g.ARCH_GAT}[arch]
    model = g.model_desc(code, dims)
    P = g.grp_param_count(model)
    parts, xs, ys, masks, opts = [], [], [], [], []
    for i, (n, E) in enumerate(sizes):
        s, d = _graph(n, E, 50 + i) if E else (torch.zeros(0, dtype=torch.int64, device=DEV),) * 2
        parts.append(g.grp_partition_from_local_coo(s, d, n))
        x, y, theta = make_inputs(n, dims, arch, 7)
        xs.append(x.to(DEV))
        ys.append(y.to(DEV))
        masks.append((torch.arange(n, device=DEV) % 3 != i % 3).to(torch.uint8) if i % 2 else None)
        opts.append(g.step_opts(estimator=g.EST_SHRINKAGE, full_graph=True, dropout_rate=dropout, dropout_seed=3, batch_id=i))
    _compare(g, parts, model, opts, xs, ys, masks, theta.to(DEV), P)


@pytest.mark.parametrize("fanouts,batches,dropout", [((5, 4, 3), [100, 7, 300], 0.5), ((2, 2, 2, 2, 2), [50, 60], 0.0), ((6,), [1, 64, 65, 200, 31], 0.0)])
def test_minibatch_steps(fanouts, batches, dropout):
    import paper_2602_01872_amd as g
    print(f"[case] merged mini-batch {fanouts} {batches}", flush=True)
    dims = [20] + [32] * (len(fanouts) - 1) + [6]
    model = g.model_desc(g.ARCH_SAGE_MEAN, dims)
    P = g.grp_param_count(model)
    parts, xs, ys, opts = [], [], [], []
    for i, b in enumerate(batches):
        n = 900 + 1700 * i
        s, d = _graph(n, 12 * n, 70 + i)
        parts.append(g.grp_partition_from_local_coo(s, d, n))
        x, y, theta = make_inputs(n, dims, "sage", 8)
        xs.append(x.to(DEV))
        ys.append(y.to(DEV))
        seeds = torch.randperm(n, generator=torch.Generator().manual_seed(i))[:b].to(torch.int32).to(DEV)
        opts.append(g.step_opts(estimator=g.EST_BATCH_MIN_DIST, full_graph=False, seeds=seeds, fanouts=fanouts, sampler_seed=4, batch_id=9,
                                dropout_rate=dropout, dropout_seed=3))
    _compare(g, parts, model, opts, xs, ys, None, theta.to(DEV), P)


def test_minibatch_steps_whose_prefix_sums_take_several_rounds():
    """Eight merged steps share a launch's waiting workgroups: blocks of up to 1.8e5 places are summed in fewer, longer parts."""
    import paper_2602_01872_amd as g
    n, fanouts, dims = 200_000, (15, 10, 5), [16, 16, 16, 6]
    model = g.model_desc(g.ARCH_SAGE_MEAN, dims)
    s, d = _graph(n, 20 * n, 90)
    part = g.grp_partition_from_local_coo(s, d, n)
    x, y, theta = make_inputs(n, dims, "sage", 8)
    opts = []
    for i in range(8):
        seeds = torch.randperm(n, generator=torch.Generator().manual_seed(i))[:1024 - i].to(torch.int32).to(DEV)
        opts.append(g.step_opts(estimator=g.EST_NONE, full_graph=False, seeds=seeds, fanouts=fanouts, sampler_seed=4, batch_id=i))
    _compare(g, [part] * 8, model, opts, [x.to(DEV)] * 8, [y.to(DEV)] * 8, None, theta.to(DEV), g.grp_param_count(model))


def _launches(g, steps):
    """Kernels that ``steps()`` launches: the nodes of a graph that it is captured in."""
    steps()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        steps()
    count = ctypes.c_size_t(0)
    assert g.binding.load().hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(count)) == 0
    return count.value


# alone: launches that each step makes by itself
@pytest.mark.parametrize("arch,dims,dropout,weighted,alone", [
    ("gcn", [32, 32, 6], 0.0, False, 0), ("gcn", [32, 32, 6], 0.5, False, 1), ("gcn_res", [32, 32, 32, 6], 0.5, False, 1),
    ("sage", [32, 32, 32, 32, 32, 6], 0.5, False, 1), ("sage", [32, 32, 200], 0.0, False, 1), ("sage", [32, 32, 6], 0.0, True, 4),
])
def test_launches_of_merged_steps(arch, dims, dropout, weighted, alone):
    import paper_2602_01872_amd as g
    print(f"[case] launches {arch} {dims} dropout={dropout} weighted={weighted}", flush=True)
    K, n = 8, 2000
    code = {"sage": g.ARCH_SAGE_MEAN, "gcn": g.ARCH_GCN, "gcn_res": g.ARCH_GCN_RESIDUAL}[arch]
    model = g.model_desc(code, dims)
    s, d = _graph(n, 12 * n, 3)
    part = g.grp_partition_weighted(s, d, torch.rand(12 * n, device=DEV) + 0.5, n, 1, 0, 0) if weighted else g.grp_partition_from_local_coo(s, d, n)
    x, y, theta = (t.to(DEV) for t in make_inputs(n, dims, arch, 7))
    opts = g.step_opts(full_graph=True, dropout_rate=dropout, dropout_seed=3)
    P = g.grp_param_count(model)
    size = g.grp_step_workspace_bytes(part, model, opts)
    ws = [torch.empty(size, dtype=torch.uint8, device=DEV) for _ in range(K)]
    grads, stats = list(torch.empty(K, P, device=DEV)), g.new_stats(K)
    recs = [stats[i * g.STATS_BYTES:(i + 1) * g.STATS_BYTES] for i in range(K)]
    one = _launches(g, lambda: g.grp_train_step(part, model, opts, x, y, None, theta, ws[0], grads[0], recs[0]))
    many = _launches(g, lambda: g.grp_train_steps([part] * K, model, [opts] * K, [x] * K, [y] * K, None, theta, ws, grads, recs))
    print(f"{one} launches of one step, {many} of {K}", flush=True)
    # what does not fit the arguments of one launch takes two or three
    assert one + (K - 1) * alone <= many <= 2 * one + (K - 1) * alone


def test_trainer_keeps_one_workspace_for_steps_that_are_not_merged():
    import paper_2602_01872_amd as g
    n = 300
    s, d = _graph(n, 900, 5)
    for arch, code, held in (("gat", g.ARCH_GAT, 1), ("gcn", g.ARCH_GCN, 3)):
        dims = [12, 16, 4]
        x, y, theta = (t.to(DEV) for t in make_inputs(n, dims, arch, 7))
        parts = [g.grp_partition_from_local_coo(s, d, n) for _ in range(3)]
        tr = g.PhaseParallelTrainer(parts, g.model_desc(code, dims), [x] * 3, [y] * 3, [None] * 3, theta, g.EST_NONE, 3)
        assert len(tr.ws) == held
        tr.run_phase([0, 1, 2])
    torch.cuda.synchronize()


def test_epochs_of_very_unequal_partitions():
    """Partitions run out of seeds one after another, so most groups have a short batch or none among them: merged and captured as one by one."""
    import paper_2602_01872_amd as g
    K, n, dims = 5, 1500, [12, 16, 16, 4]
    s, d = _graph(n, 9 * n, 6)
    part = g.grp_partition_from_local_coo(s, d, n)
    x, y, theta = (t.to(DEV) for t in make_inputs(n, dims, "sage", 7))
    masks = [(torch.arange(n, device=DEV) < count).to(torch.uint8) for count in (37, 1000, 64, 0, 500)]
    model = g.model_desc(g.ARCH_SAGE_MEAN, dims)
    runs = []
    for lanes, graphs in ((1, False), (4, False), (4, True), (5, True)):
        tr = g.MiniBatchTrainer([part] * K, model, [x] * K, [y] * K, masks, theta, g.EST_SHRINKAGE, K, 64, (4, 3, 5), 21,
                                g.optimizer_desc(g.OPT_ADAM, lr=0.003), dropout_rate=0.3, dropout_seed=2, lanes=lanes, graphs=graphs)
        for _ in range(2):
            tr.run_epoch()
        torch.cuda.synchronize()
        runs.append((tr.theta.clone(), tr.losses()))
    assert len(runs[0][1]) == 2 * 16
    for theta_, losses in runs[1:]:
        assert torch.equal(theta_, runs[0][0]) and losses == runs[0][1]


def _compare(g, parts, model, opts, xs, ys, masks, theta, P):
    K = len(parts)
    size = max(g.grp_step_workspace_bytes(p, model, o) for p, o in zip(parts, opts))
    ws = [torch.full((size,), 3 + i, dtype=torch.uint8, device=DEV) for i in range(K)]
    ld = (P + 3) // 4 * 4
    one, many = torch.full((K, ld), 9.0, device=DEV), torch.full((K, ld), 9.0, device=DEV)
    st1, stm = g.new_stats(K), g.new_stats(K)
    cut = lambda t, i: t[i * g.STATS_BYTES:(i + 1) * g.STATS_BYTES]
    for i in range(K):
        g.grp_train_step(parts[i], model, opts[i], xs[i], ys[i], masks[i] if masks else None, theta, ws[0], one[i], cut(st1, i))
    for _ in range(2):
        g.grp_train_steps(parts, model, opts, xs, ys, masks, theta, ws, list(many), [cut(stm, i) for i in range(K)])
    torch.cuda.synchronize()
    assert torch.equal(st1, stm)
    assert torch.equal(one, many)
