"""The transposed blocks of a mini-batch step at the edges of the sort that builds them: rows of 127 to 129 edges (ranked / counted), more
edges than one round of LDS holds, rows shared by more destinations than one round counts.  A gradient that went through a wrongly
transposed block is wrong, and a row left in order of arrival changes the bits from run to run."""
import pytest
import torch

from oracle import graph as ograph
from oracle import step as ostep
from tests._cases import TOL_FP32, assert_step_grads_close, make_inputs

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("n_seeds,shared", [(127, 1), (128, 1), (129, 1), (700, 40), (8193, 3), (9000, 200)])
def test_sources_shared_by_many_seeds(n_seeds, shared):
    import paper_2602_01872_amd as g
    print(f"[case] transposed n_seeds={n_seeds} shared={shared}", flush=True)
    n = n_seeds + shared
    gen = torch.Generator().manual_seed(n)
    dst = torch.arange(n_seeds).repeat_interleave(4)            # every seed draws from the same few nodes, some of them twice
    src = n_seeds + torch.randint(shared, (dst.numel(),), generator=gen)
    src = torch.cat([src, torch.randint(n_seeds, (shared,), generator=gen)])
    dst = torch.cat([dst, n_seeds + torch.arange(shared)])
    want = ograph.local_graph_from_edges(src.numpy(), dst.numpy(), n)
    part = g.grp_partition_from_local_coo(src.to(DEV), dst.to(DEV), n)
    dims, fanouts = [8, 12, 5], (2, 3)
    x, y, theta = make_inputs(n, dims, "sage", 3)
    seeds = torch.randperm(n_seeds, generator=gen).to(torch.int32)
    opts = g.step_opts(estimator=g.EST_SHRINKAGE, full_graph=False, seeds=seeds.to(DEV), fanouts=fanouts, sampler_seed=5, batch_id=2)
    model = g.model_desc(g.ARCH_SAGE_MEAN, dims)
    ws = torch.empty(g.grp_step_workspace_bytes(part, model, opts), dtype=torch.uint8, device=DEV)
    P = g.grp_param_count(model)
    grads = []
    for fill in (0, 255, 7):
        ws.fill_(fill)
        grad, st = torch.zeros(P, device=DEV), g.new_stats(1)
        g.grp_train_step(part, model, opts, x.to(DEV), y.to(DEV), None, theta.to(DEV), ws, grad, st)
        grads.append(grad)
    assert torch.equal(grads[0], grads[1]) and torch.equal(grads[0], grads[2])
    mb = dict(seeds=seeds.numpy(), fanouts=fanouts, sampler_seed=5, batch_id=2)

    def oracle_fn(relu_flip=None, near_kink=None):
        return ostep.train_step(want, "sage", dims, theta.double().numpy(), x.double().numpy(), y.numpy(), estimator=3, minibatch=mb,
                                relu_flip=relu_flip, near_kink=near_kink)
    assert_step_grads_close(grads[0].cpu().numpy(), oracle_fn, "sage", dims, TOL_FP32)
