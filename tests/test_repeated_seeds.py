"""A seed list may name a node more than once: seeds outside the partition are replaced by node 0, and that seeds are distinct is not
checked.  The sampled blocks then hold more sources than the partition has nodes, and every array is sized for them."""
import ctypes as C
import os

import numpy as np
import pytest
import torch

import paper_2602_01872_amd as g
import synth

DEV = "cuda:0"
MOST = 16


class Bounds(C.Structure):
    _fields_ = [("dst", C.c_int64 * MOST), ("nnz", C.c_int64 * MOST), ("src", C.c_int64 * MOST)]


@pytest.mark.parametrize("n,n_seeds,distinct,degree", [(10, 20, 3, 4), (10, 10, 5, 9), (200, 150, 100, 40), (200, 150, 1, 40), (50, 7, 7, 49), (300, 2, 1, 3)])
def test_bounds_hold_for_repeated_seeds(n, n_seeds, distinct, degree):
    if not os.path.exists(g.LIB_PATH):
        import __graft_entry__
        __graft_entry__.build()
    fn = getattr(g.load(), "_ZN3grp14sampler_boundsEllPKiiPNS_13SamplerBoundsE")
    fn.argtypes, fn.restype = [C.c_int64, C.c_int64, C.POINTER(C.c_int32), C.c_int, C.c_void_p], None
    fanouts = (C.c_int32 * 3)(64, 64, 64)                    # (every neighbour)
    b = Bounds()
    fn(n, n_seeds, fanouts, 3, C.addressof(b))
    dst = [i % distinct for i in range(n_seeds)]
    for l in (2, 1, 0):
        assert len(dst) <= b.dst[l] and len(dst) * degree <= b.nnz[l]
        reached = {(v + j) % n for v in set(dst) for j in range(1, degree + 1)}
        dst = dst + sorted(reached - set(dst))
        if l > 0:
            assert len(dst) <= b.src[l], l


@pytest.mark.gpu
@pytest.mark.parametrize("n,n_seeds,good", [(10, 20, 4), (200, 150, 100), (2_000, 1_999, 500)])
def test_step_with_seeds_outside_the_partition(n, n_seeds, good):
    s, d = synth.uniform_graph(n, 40 * n, seed=3, device=DEV)
    part = g.grp_partition(s, d, n, 1, 0, 0)
    dims, fanouts = [12, 16, 16, 5], (15, 10, 5)
    model = g.model_desc(g.ARCH_SAGE_MEAN, dims)
    theta = synth.model_weights("sage", dims, 1).to(DEV)
    x, y = synth.normal_matrix(n, dims[0], 1).to(DEV), synth.labels(n, dims[-1], 1).to(DEV)
    P = g.grp_param_count(model)

    def step(seeds):
        seeds = torch.tensor(seeds, dtype=torch.int32, device=DEV)
        opts = g.step_opts(full_graph=False, seeds=seeds, fanouts=fanouts, sampler_seed=1, batch_id=1)
        size, guard = g.grp_step_workspace_bytes(part, model, opts), 1 << 16
        ws = torch.full((size + guard,), 0x5A, dtype=torch.uint8, device=DEV)
        grad, stats = torch.zeros(P, device=DEV), g.new_stats(1)
        g.grp_train_step(part, model, opts, x, y, None, theta, ws[:size], grad, stats)
        assert bool((ws[size:] == 0x5A).all())
        for l in range(3):
            b = g.binding.read_block(part, model, opts, ws[:size], l)
            assert b["rowptr"][-1] == b["col"].size and np.all(np.diff(b["rowptr"]) >= 0)
            assert b["col"].size == 0 or (0 <= b["col"].min() and b["col"].max() < (n if l == 0 else b["src_nodes"].size))
        return grad, g.read_stats(stats)[0]
    before, _ = step(range(good))
    _, st = step([*range(good), *[n + 5] * (n_seeds - good)])
    assert int(st["nnz_used"]) == good - n_seeds
    _, st = step([*range(good), *[0] * (n_seeds - good)])    # (repeated by the caller)
    assert int(st["nnz_used"]) > 0 and int(st["S"]) == n_seeds
    after, _ = step(range(good))
    assert torch.equal(before, after)
    part.destroy()
