"""The loss kernels at the class counts where they change (registers for up to 192 classes, memory above) and at row counts of
one and a few workgroups, against the oracle; and a mini-batch step on workspaces that hold anything at all: the sampler's node map is
never cleared, so what it held before must not show in a single bit."""
import numpy as np
import pytest
import torch

import synth
from oracle import graph as ograph
from oracle import step as ostep
from tests._cases import TOL_FP32, assert_step_grads_close

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.fixture(scope="module")
def g():
    import paper_2602_01872_amd as lib
    lib.load()
    return lib


@pytest.mark.parametrize("N,C", [(1, 65), (15, 128), (17, 129), (255, 172), (257, 192), (400, 193), (4097, 100)])
def test_loss_at_class_and_row_edges(g, N, C):
    dims, seed = [6, C], 5
    s, d = synth.uniform_graph(N, 4 * N, seed=seed)
    part = g.grp_partition(s.to(DEV), d.to(DEV), N, 1, seed, 0)
    op = ograph.partition(s.numpy(), d.numpy(), N, 1, seed, 0)
    x, y, theta = synth.normal_matrix(N, 6, seed), synth.labels(N, C, seed), synth.model_weights("sage", dims, seed)
    model, opts = g.model_desc(g.ARCH_SAGE_MEAN, dims), g.step_opts(full_graph=True)
    ws = torch.empty(g.grp_step_workspace_bytes(part, model, opts), dtype=torch.uint8, device=DEV)
    grad, stats = torch.full((g.grp_param_count(model),), float("nan"), device=DEV), g.new_stats(1)
    g.grp_train_step(part, model, opts, x.to(DEV), y.to(DEV), None, theta.to(DEV), ws, grad, stats)
    torch.cuda.synchronize()

    def oracle(**kw):
        return ostep.train_step(op, "sage", dims, theta.double().numpy(), x.double().numpy(), y.numpy(), **kw)
    _, want = assert_step_grads_close(grad.cpu().numpy(), oracle, "sage", dims, TOL_FP32)
    got = g.read_stats(stats)[0]
    assert int(got["S"]) == want["S"] and float(got["R"]) == want["R"]
    assert abs(float(got["loss"]) - want["loss"]) <= TOL_FP32 * abs(want["loss"])
    assert np.isclose(float(got["sum_ratio"]), want["sum_ratio"], rtol=1e-12)


@pytest.mark.parametrize("fill", [1, 7, -1, 2_000_000_000])
def test_minibatch_step_on_a_used_workspace(g, fill):
    N, E, dims, seed = 5000, 60_000, [12, 16, 16, 5], 3
    s, d = synth.rmat_graph(13, E, seed=seed, n_nodes=N)
    part = g.grp_partition(s.to(DEV), d.to(DEV), N, 1, seed, 0)
    x, y, theta = synth.normal_matrix(N, 12, seed).to(DEV), synth.labels(N, 5, seed).to(DEV), synth.model_weights("sage", dims, seed).to(DEV)
    seeds = torch.randperm(N, generator=torch.Generator().manual_seed(1))[:300].to(torch.int32)
    seeds[7] = seeds[3]                                    # a seed may be given twice
    model = g.model_desc(g.ARCH_SAGE_MEAN, dims)
    opts = g.step_opts(full_graph=False, seeds=seeds.to(DEV), fanouts=[4, 4, 4], sampler_seed=9)
    bytes_ = g.grp_step_workspace_bytes(part, model, opts)
    out = []
    for value in (0, fill):
        ws = torch.full(((bytes_ + 3) // 4,), value, dtype=torch.int32, device=DEV).view(torch.uint8)
        grad, stats = torch.zeros(g.grp_param_count(model), device=DEV), g.new_stats(1)
        for _ in range(2):                                 # the second pass finds the first one's map
            g.grp_train_step(part, model, opts, x, y, None, theta, ws, grad, stats)
            out.append((grad.clone(), stats.clone()))
    torch.cuda.synchronize()
    for grad, stats in out[1:]:
        assert torch.equal(grad, out[0][0]) and torch.equal(stats, out[0][1])


@pytest.mark.parametrize("arch,N,dims", [
    ("sage", 700, [33, 31, 65, 97]), ("sage", 26_000, [129, 95, 33, 32]), ("gcn", 26_000, [31, 129, 97, 63]), ("gcn", 700, [127, 64, 1, 3])])
def test_weights_at_tile_edges_on_a_used_workspace(g, arch, N, dims):
    """The products read the weights from tiles of 32 k by up to 128 rows that the step writes itself: one column past a tile and one short
    of it, side by side and alone, 64-row and 128-row products; what the workspace held before (NaN) must not show."""
    seed = 11
    s, d = synth.uniform_graph(N, 2 * N, seed=seed)
    part = g.grp_partition(s.to(DEV), d.to(DEV), N, 1, seed, 0)
    op = ograph.partition(s.numpy(), d.numpy(), N, 1, seed, 0)
    x, y, theta = synth.normal_matrix(N, dims[0], seed), synth.labels(N, dims[-1], seed), synth.model_weights(arch, dims, seed)
    model, opts = g.model_desc(g.ARCH_SAGE_MEAN if arch == "sage" else g.ARCH_GCN, dims), g.step_opts(full_graph=True)
    ws = torch.full((g.grp_step_workspace_bytes(part, model, opts),), 255, dtype=torch.uint8, device=DEV)
    grad, stats = torch.full((g.grp_param_count(model),), float("nan"), device=DEV), g.new_stats(1)
    g.grp_train_step(part, model, opts, x.to(DEV), y.to(DEV), None, theta.to(DEV), ws, grad, stats)
    torch.cuda.synchronize()

    def oracle(**kw):
        return ostep.train_step(op, arch, dims, theta.double().numpy(), x.double().numpy(), y.numpy(), **kw)
    assert_step_grads_close(grad.cpu().numpy(), oracle, arch, dims, TOL_FP32)


@pytest.mark.parametrize("arch,N,dims", [
    ("gcn", 300, [7, 5, 6, 9, 3]), ("gcn", 900, [33, 64, 31, 32, 16]), ("gcn", 5000, [64, 128, 8, 130, 41, 5]), ("sage", 5000, [12] * 8 + [3]),
    ("gcn", 50_001, [20, 130, 96, 61, 33, 7]), ("gcn", 700, [16, 20, 193])])
def test_sums_that_a_deep_step_leaves_to_its_end(g, arch, N, dims):
    """Every layer's products and column sums leave partial results to the step's last launch: more of them than three layers have, of few and
    of many slices, in vectors and not, column sums from the loss (up to 192 classes) and from products of 64 and of
    128 rows; one step alone and two that share their launches, on workspaces that held NaN."""
    seed = 13
    s, d = synth.rmat_graph(13, 6 * N, seed=seed, n_nodes=N)
    part = g.grp_partition(s.to(DEV), d.to(DEV), N, 1, seed, 0)
    op = ograph.partition(s.numpy(), d.numpy(), N, 1, seed, 0)
    x, y, theta = synth.normal_matrix(N, dims[0], seed), synth.labels(N, dims[-1], seed), synth.model_weights(arch, dims, seed)
    model, opts = g.model_desc(g.ARCH_SAGE_MEAN if arch == "sage" else g.ARCH_GCN, dims), g.step_opts(full_graph=True)
    bytes_, P = g.grp_step_workspace_bytes(part, model, opts), g.grp_param_count(model)
    xd, yd, td, out = x.to(DEV), y.to(DEV), theta.to(DEV), []
    for count in (1, 2):
        ws = [torch.full((bytes_,), 255, dtype=torch.uint8, device=DEV) for _ in range(count)]
        grads, stats = [torch.full((P,), float("nan"), device=DEV) for _ in range(count)], [g.new_stats(1) for _ in range(count)]
        g.grp_train_steps([part] * count, model, [opts] * count, [xd] * count, [yd] * count, None, td, ws, grads, stats)
        out += list(zip(grads, stats))
    torch.cuda.synchronize()
    for grad, stat in out[1:]:
        assert torch.equal(grad, out[0][0]) and torch.equal(stat, out[0][1])

    def oracle(**kw):
        return ostep.train_step(op, arch, dims, theta.double().numpy(), x.double().numpy(), y.numpy(), **kw)
    assert_step_grads_close(out[0][0].cpu().numpy(), oracle, arch, dims, TOL_FP32)
