"""Rows packed without padding (pitch = width, base at any element): neighbour sums and both GEMM directions read the last,
partial vector of a row moved back to the row's end.  Widths around the vector and tile edges, fp32 and bf16 operands, against
float64; NaN behind the last row would show a read past it that reached a result."""
import numpy as np
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


def packed(rows, cols, dtype, off, seed):
    """[rows x cols] without padding, `off` elements into an allocation that holds NaN elsewhere; and its values."""
    buf = torch.full((off + rows * cols + 8,), float("nan"), device=DEV, dtype=dtype)
    v = buf[off:off + rows * cols].view(rows, cols)
    v.copy_(synth.normal_matrix(rows, cols, seed))
    return buf, v, v.double().cpu()


def close(got, want, tol):
    got, want = got.double().cpu(), want
    assert torch.isfinite(got).all()
    assert float((got - want).abs().max() / want.abs().max()) <= tol


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("F", [1, 3, 4, 5, 7, 31, 33, 75, 130, 257])
def test_packed_rows(g, F, dtype):
    code = g.DTYPE_BF16 if dtype == torch.bfloat16 else g.DTYPE_FP32
    n, off = 3000, F % 3
    # neighbour sums, both directions, with rows long enough to be split
    s, d = synth.rmat_graph(12, 60000, seed=F, n_nodes=n)
    s[:6000] = 5
    d[6000:12000] = 7
    part = g.grp_partition(s.to(DEV), d.to(DEV), n, 1, 1, 0)
    _, X, Xh = packed(n, F, dtype, off, F)
    for transposed in (False, True):
        Y = torch.full((n, F), float("nan"), device=DEV)
        g.grp_spmm(part, transposed, g.SCALE_MEAN, True, F, X, F, code, Y, F)
        a, b = (d, s) if transposed else (s, d)
        deg = torch.bincount(b, minlength=n).double().clamp(min=1)
        want = (torch.zeros(n, F, dtype=torch.float64).index_add_(0, b, Xh[a]) + Xh) / deg[:, None]
        close(Y, want, 1e-5)
    # X W^T and X^T D
    M, N = 1037, 96
    W = synth.normal_matrix(N, (F + 3) // 4 * 4, F + 1).to(DEV)
    C = torch.full((M, N), float("nan"), device=DEV)
    g.grp_gemm_nt(M, N, F, X[:M], F, code, W, W.shape[1], C, N)
    close(C, Xh[:M] @ W[:, :F].double().cpu().T, 1e-5)
    for Nd in (3, 41, 130):
        _, D, Dh = packed(M, Nd, torch.float32, 1, F + 2)
        ws = torch.empty(max(g.grp_gemm_tn_workspace_bytes(M, F, Nd), 16), dtype=torch.uint8, device=DEV)
        C = torch.full((F, Nd), float("nan"), device=DEV)
        g.grp_gemm_tn(M, F, Nd, X[:M], F, code, D, Nd, C, Nd, ws)
        close(C, Xh[:M].T @ Dh, 1e-5)
