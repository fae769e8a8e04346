"""The scratch that a transposed product asks for covers every product of fewer rows: a mini-batch step sizes it once per layer, by the larger
of the layer's two row counts, and launches products over the smaller one with it."""
import os

import numpy as np
import pytest
import torch

import paper_2602_01872_amd as g
import synth

DEV = "cuda:0"
SHAPES = [(128, 128), (100, 256), (256, 256), (256, 47), (64, 64), (128, 40), (16, 8), (300, 130), (1024, 1024)]


@pytest.mark.parametrize("K,N", SHAPES)
def test_scratch_does_not_shrink_as_rows_grow(K, N):
    if not os.path.exists(g.LIB_PATH):
        import __graft_entry__
        __graft_entry__.build()
    rows = sorted({*range(1, 20_000, 31), *(2 ** i + d for i in range(5, 26) for d in (-1, 0, 1)), 10_584, 6_000, 8_192, 11_904})
    need = [g.grp_gemm_tn_workspace_bytes(m, K, N) for m in rows]
    assert all(a <= b for a, b in zip(need, need[1:]))


@pytest.mark.gpu
@pytest.mark.parametrize("K,N", [(128, 128), (256, 47), (64, 64)])
def test_products_of_fewer_rows_run_in_the_scratch_of_more(K, N):
    most = 10_584
    ws = torch.empty(max(g.grp_gemm_tn_workspace_bytes(most, K, N), 16), dtype=torch.uint8, device=DEV)
    a, b = synth.normal_matrix(most, K, 3), synth.normal_matrix(most, N, 4)
    ad, bd = a.to(DEV), b.to(DEV)
    for m in (1, 33, 2_048, 2_049, 4_096, 6_000, 8_192, 8_193, most):
        c = torch.empty(K, N, device=DEV)
        g.grp_gemm_tn(m, K, N, ad, K, g.DTYPE_FP32, bd, N, c, N, ws)
        want = a[:m].double().T @ b[:m].double()
        # products of two N(0, 1): the sizes of m of them add up to 0.64 m, and fp32 arithmetic keeps a sum within a few 2^-23 of that
        assert float((c.cpu().double() - want).abs().max()) <= 8 * 2.0 ** -23 * m


# The sampled blocks of these steps have a layer with more inputs than outputs, whose product over the outputs is cut into more slices than
# one over the inputs (1000 seeds: 6000 rows in 94 slices, 10 584 in 83).
@pytest.mark.gpu
@pytest.mark.parametrize("n,batch,fanouts,dims", [
    (10_584, 1_000, (15, 10, 5), [128, 128, 128, 40]), (10_000, 1_000, (15, 10, 5), [128, 128, 128, 40]),
    (8_193, 1_024, (15, 10, 5), [128, 128, 128, 40]), (2_500, 256, (15, 10, 5), [100, 256, 256, 47]),
    (4_097, 512, (15, 10, 5), [128, 128, 128, 40]), (12_160, 1_024, (5, 10, 15), [128, 256, 256, 40])])
def test_minibatch_step_runs_in_the_workspace_it_asks_for(n, batch, fanouts, dims):
    s, d = synth.uniform_graph(n, 8 * n, seed=n, device=DEV)
    part = g.grp_partition(s, d, n, 1, 0, 0)
    model = g.model_desc(g.ARCH_SAGE_MEAN, dims)
    theta = synth.model_weights("sage", dims, 1).to(DEV)
    x, y = synth.normal_matrix(n, dims[0], 1).to(DEV), synth.labels(n, dims[-1], 1).to(DEV)
    seeds = torch.empty(n, dtype=torch.int32, device=DEV)
    assert g.grp_epoch_seeds(part, None, 1, 0, seeds) == n
    opts = g.step_opts(full_graph=False, seeds=seeds[:batch], fanouts=fanouts, sampler_seed=1, batch_id=1)
    P = g.grp_param_count(model)
    bytes_ = g.grp_step_workspace_bytes(part, model, opts)

    def step(extra):
        grad, stats = torch.full((P,), float("nan"), device=DEV), g.new_stats(1)
        g.grp_train_step(part, model, opts, x, y, None, theta, torch.empty(bytes_ + extra, dtype=torch.uint8, device=DEV), grad, stats)
        return grad.cpu().numpy(), g.read_stats(stats)[0]
    (tight, st), (roomy, st2) = step(0), step(1 << 20)
    assert int(st["S"]) == batch and np.isfinite(tight).all() and np.abs(tight).max() > 0
    assert np.array_equal(tight, roomy) and st == st2
    part.destroy()
