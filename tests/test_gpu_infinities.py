"""Infinite operands: an infinity times a finite number stays infinite, in neighbour sums and in dense products, and nothing that it
does not enter changes."""
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.fixture(scope="module")
def g():
    import paper_2602_01872_amd as lib
    lib.load()
    return lib


def same_kind(got, want):
    """The same infinities and NaNs at the same places."""
    got, want = got.double().cpu(), want.double().cpu()
    assert torch.equal(torch.isnan(got), torch.isnan(want))
    assert torch.equal(torch.isinf(got), torch.isinf(want))
    assert torch.equal(torch.sign(got[torch.isinf(got)]), torch.sign(want[torch.isinf(want)]))
    fin = torch.isfinite(want)
    assert float((got[fin] - want[fin]).abs().max() / want[fin].abs().max()) <= 1e-5


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("F", [1, 3, 4, 8, 13, 16, 32, 47, 64, 100, 130, 256])
def test_neighbour_sums(g, F, dtype):
    """Rows of 0 to 40 neighbours, so that batches of every width end at every place, some with an infinite last neighbour."""
    n = 2000
    dst = torch.repeat_interleave(torch.arange(n), torch.arange(n) % 41)
    src = torch.randint(n, (dst.numel(),), generator=torch.Generator().manual_seed(F))
    X = synth.normal_matrix(n, F, F).to(dtype)
    X[n - 30:] = float("inf")                                # a row's sources ascend: these are the last of the rows that have them
    X[n - 10:] = float("-inf")
    part = g.grp_partition(src.to(DEV), dst.to(DEV), n, 1, 1, 0)
    Y = torch.full((n, F), float("nan"), device=DEV)
    g.grp_spmm(part, False, g.SCALE_NONE, False, F, X.to(DEV).contiguous(), F, g.DTYPE_BF16 if dtype == torch.bfloat16 else g.DTYPE_FP32, Y, F)
    same_kind(Y, torch.zeros(n, F, dtype=torch.float64).index_add_(0, dst, X.double()[src]))
