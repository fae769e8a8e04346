"""Dense products over at least 65,409 rows take the weights as bf16 planes made once per product: full-graph steps at the smallest
such size against the oracle, at widths around the edges of the 64-, 96- and 128-column tiles and of the 32-deep k-tiles, with tight
and bf16 feature rows and with two products in one launch."""
import numpy as np
import pytest
import torch

import synth
from oracle import graph as ograph
from oracle import step as ostep
from tests._cases import TOL_FP32, assert_step_grads_close

pytestmark = pytest.mark.gpu
DEV = "cuda"
ARCH = {"sage": 0, "gcn": 1, "gat": 3}


@pytest.fixture(scope="module")
def g():
    import paper_2602_01872_amd as lib
    lib.load()
    return lib


@pytest.mark.parametrize("arch,dims,bf16", [
    ("sage", [33, 70, 130, 9], False),
    ("sage", [75, 128, 47], True),
    ("sage", [64, 129, 97, 64], True),
    ("gcn", [96, 65, 12], False),
    ("gat", [31, 92, 20], False),
])
def test_steps_over_many_rows(g, arch, dims, bf16):
    N, E, seed = 65_537, 200_000, 11
    s, d = synth.rmat_graph(17, E, seed=seed, n_nodes=N)
    part = g.grp_partition(s.to(DEV), d.to(DEV), N, 1, seed, 0)
    op = ograph.partition(s.numpy(), d.numpy(), N, 1, seed, 0)
    x = synth.normal_matrix(N, dims[0], seed)
    if bf16:
        x = synth.to_bf16_rne(x)
    y = synth.labels(N, dims[-1], seed)
    theta = synth.model_weights(arch, dims, seed)
    model = g.model_desc(ARCH[arch], dims, g.DTYPE_BF16 if bf16 else g.DTYPE_FP32)
    opts = g.step_opts(full_graph=True)
    ws = torch.empty(g.grp_step_workspace_bytes(part, model, opts), dtype=torch.uint8, device=DEV)
    grad = torch.full((g.grp_param_count(model),), float("nan"), device=DEV)
    stats = g.new_stats(1)
    g.grp_train_step(part, model, opts, x.to(DEV), y.to(DEV), None, theta.to(DEV), ws, grad, stats)
    torch.cuda.synchronize()
    assert np.isfinite(grad.cpu().numpy()).all()

    def oracle(**kw):
        return ostep.train_step(op, arch, dims, theta.double().numpy(), x.double().numpy(), y.numpy(), **kw)
    assert_step_grads_close(grad.cpu().numpy(), oracle, arch, dims, TOL_FP32)
