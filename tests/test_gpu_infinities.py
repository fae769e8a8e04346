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
    assert not fin.any() or float((got[fin] - want[fin]).abs().max() / want[fin].abs().max()) <= 1e-5


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


def with_infinities(rows, cols, dtype, seed, pitch=None):
    """Normal deviates with single infinities of both signs, one row with two of opposite sign, and a NaN, in a matrix of `pitch`
    columns; and its values in float64."""
    x = synth.normal_matrix(rows, cols, seed).to(dtype)
    x[1, 0], x[rows // 2, cols // 2], x[rows - 1, cols - 1] = float("inf"), float("-inf"), float("inf")
    x[2, 0], x[2, cols - 1] = float("inf"), float("-inf")
    if rows > 6:
        x[5, cols // 3] = float("nan")
    buf = torch.zeros(rows, pitch or cols, dtype=dtype)
    buf[:, :cols] = x
    return buf.to(DEV), x.double()


def product(a, b):
    """a @ b of float64 matrices, infinities included, without sums that meet 0 x infinity."""
    return (a[:, :, None] * b[None, :, :]).sum(1)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("N,K", [(3, 4), (40, 5), (64, 36), (70, 33), (100, 64), (130, 75), (260, 32)])
def test_dense_products(g, N, K, dtype):
    code = g.DTYPE_BF16 if dtype == torch.bfloat16 else g.DTYPE_FP32
    for M in (65, 300):
        A, Ah = with_infinities(M, K, dtype, K)
        W, Wh = with_infinities(N, K, torch.float32, N, (K + 3) // 4 * 4)
        if M == 300:                                         # once with finite weights
            W, Wh = torch.nan_to_num(W, 1.0, 1.0, 1.0), torch.nan_to_num(Wh, 1.0, 1.0, 1.0)
        C = torch.full((M, N), 7.0, device=DEV)
        g.grp_gemm_nt(M, N, K, A, K, code, W, W.shape[1], C, N)
        same_kind(C, product(Ah, Wh.T))
        D = synth.normal_matrix(M, N, N + 1)
        ws = torch.empty(max(g.grp_gemm_tn_workspace_bytes(M, K, N), 16), dtype=torch.uint8, device=DEV)
        C = torch.full((K, N), 7.0, device=DEV)
        g.grp_gemm_tn(M, K, N, A, K, code, D.to(DEV), N, C, N, ws)
        same_kind(C, torch.stack([(Ah[:, k, None] * D.double()).sum(0) for k in range(K)]))


@pytest.mark.parametrize("dims", [[36, 70, 9], [33, 130, 20]])
def test_activations_over_many_rows(g, dims):
    """Products over at least 65,409 rows take the weights as planes made once: an infinite feature leaves infinities of the weights'
    signs, of which ReLU keeps the positive ones."""
    N, E, seed = 65_537, 120_000, 3
    s, d = synth.rmat_graph(17, E, seed=seed, n_nodes=N)
    part = g.grp_partition(s.to(DEV), d.to(DEV), N, 1, seed, 0)
    x = synth.normal_matrix(N, dims[0], seed)
    odd = torch.arange(7, N, 997)
    keep = ~torch.isin(d, odd)                                # their neighbourhoods stay finite: rows that gather no odd row
    x[odd, 5] = float("inf")
    theta = synth.model_weights("sage", dims, seed)
    model = g.model_desc(g.ARCH_SAGE_MEAN, dims)
    opts = g.step_opts(full_graph=True)
    part = g.grp_partition(s[keep].to(DEV), d[keep].to(DEV), N, 1, seed, 0)
    ws = torch.empty(g.grp_step_workspace_bytes(part, model, opts), dtype=torch.uint8, device=DEV)
    grad = torch.empty(g.grp_param_count(model), device=DEV)
    g.grp_train_step(part, model, opts, x.to(DEV), synth.labels(N, dims[-1], seed).to(DEV), None, theta.to(DEV), ws, grad, g.new_stats(1))
    torch.cuda.synchronize()
    w_self = theta[:dims[0] * dims[1]].view(dims[0], dims[1])
    want = torch.where(w_self[5] > 0, float("inf"), 0.0)
    rr = odd.repeat_interleave(dims[1]).numpy()
    cc = torch.arange(dims[1]).repeat(odd.numel()).numpy()
    got = torch.as_tensor(g.read_activation(part, model, opts, ws, 0, rr, cc)).view(odd.numel(), dims[1])
    assert torch.equal(got, want.expand_as(got).to(got.dtype))


@pytest.mark.parametrize("K", [1, 40])
def test_largest_floats(g, K):
    """Numbers whose first bf16 would round up to infinity, and sums of planes that pass the largest float, keep their finite products."""
    M, N, big = 70, 24, torch.finfo(torch.float32).max
    A = torch.zeros(M, (K + 3) // 4 * 4, device=DEV)
    A[:, 0] = torch.tensor([big, -big, big * (1 - 2.0 ** -20), 1.0, 1e30, -1e-30, 2.0 ** 127], device=DEV).repeat(10)
    W = torch.zeros(N, A.shape[1], device=DEV)
    W[:, 0] = torch.tensor([1.0, -1.0, 0.5, 1 / 3], device=DEV).repeat(6)
    want = A[:, :1].double() * W[:, 0].double()[None, :]
    C = torch.full((M, N), 7.0, device=DEV)
    g.grp_gemm_nt(M, N, K, A, A.shape[1], g.DTYPE_FP32, W, W.shape[1], C, N)
    assert float(((C.double() - want) / want).abs().max()) <= 2.0 ** -23
    B = torch.zeros(4, N, device=DEV)                        # A^T B over four rows, one of them not zero
    B[2] = W[:, 0]
    X = torch.zeros(4, M, device=DEV)
    X[2] = A[:, 0]
    ws = torch.empty(max(g.grp_gemm_tn_workspace_bytes(4, M, N), 16), dtype=torch.uint8, device=DEV)
    C = torch.full((M, N), 7.0, device=DEV)
    g.grp_gemm_tn(4, M, N, X, M, g.DTYPE_FP32, B, N, C, N, ws)
    assert float(((C.double() - want) / want).abs().max()) <= 2.0 ** -23
