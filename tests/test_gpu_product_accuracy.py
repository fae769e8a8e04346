"""How accurate the dense products are, against float64: NT and TN take fp32 operands as sums of three bf16 numbers, and have to be
at least as good as fp32 arithmetic at every length."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda"
U = 2.0 ** -24                 # half a unit in the last place, relative to a number's power of two
ROUND = 0.45 * U               # rms relative error of one rounding (uniform error, mantissas spread over a binade)


@pytest.fixture(scope="module")
def g():
    import paper_2602_01872_amd as lib
    lib.load()
    return lib


def values(kind, rows, cols, seed):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    if kind == "normal":
        return torch.randn(rows, cols, generator=gen, device=DEV)
    if kind == "uniform":
        return torch.rand(rows, cols, generator=gen, device=DEV) + 2.0 ** -20
    return torch.full((rows, cols), 1 / 3, device=DEV)


def nt(g, A, B):
    """(A B^T, float64 reference)"""
    M, K = A.shape
    N, Kp = B.shape[0], (K + 3) // 4 * 4
    Ap, Bp = torch.zeros(M, Kp, device=DEV, dtype=A.dtype), torch.zeros(N, Kp, device=DEV)
    Ap[:, :K], Bp[:, :K] = A, B
    C = torch.empty(M, N, device=DEV)
    g.grp_gemm_nt(M, N, K, Ap, Kp, g.DTYPE_BF16 if A.dtype == torch.bfloat16 else g.DTYPE_FP32, Bp, Kp, C, N)
    return C.double(), A.double() @ B.double().T


def tn(g, A, B):
    """(A^T B, float64 reference)"""
    (M, K), N = A.shape, B.shape[1]
    ws = torch.empty(max(g.grp_gemm_tn_workspace_bytes(M, K, N), 16), dtype=torch.uint8, device=DEV)
    C = torch.empty(K, N, device=DEV)
    g.grp_gemm_tn(M, K, N, A, K, g.DTYPE_BF16 if A.dtype == torch.bfloat16 else g.DTYPE_FP32, B, N, C, N, ws)
    want = torch.zeros(K, N, device=DEV, dtype=torch.float64)
    for lo in range(0, M, 100_000):
        want += A[lo:lo + 100_000].double().T @ B[lo:lo + 100_000].double()
    return C.double(), want


def rms(x):
    return float(x.pow(2).mean().sqrt())


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("way", ["nt", "tn"])
def test_one_term_is_rounded_once(g, way, bf16):
    """A product of two numbers is exact before its one rounding (a 1/64 of it is left for the cuts of the small terms)."""
    A, B = values("uniform", 5000 if way == "nt" else 128, 1, 1), values("normal", 120, 1, 2)
    if way == "tn":
        A, B = A.T.contiguous(), B.T.contiguous()
    if bf16:
        A = A.bfloat16()
    got, want = (nt if way == "nt" else tn)(g, A, B)
    assert float(((got - want) / want).abs().max()) <= U * (1 + 1 / 64)


@pytest.mark.parametrize("kinds", [("normal", "normal"), ("uniform", "third"), ("uniform", "uniform")])
@pytest.mark.parametrize("way", ["nt", "tn"])
@pytest.mark.parametrize("n", [2, 3, 4, 8, 17, 32, 33, 64, 100, 256, 512, 1024])
def test_rounding_of_sums(g, way, kinds, n):
    """Sums of n terms.  A tile of 32 terms is rounded when each eight of its products are added and when its two parts are:
    five times, the early ones at a smaller sum; the running sum once a tile, on average at 1/sqrt(2) of its final size.  (A TN
    product over more than 128 rows is cut into slices, whose sums are added in fp32 as well: no more roundings in all.)"""
    tiles = math.ceil(n / 32)
    bound = 1.25 * ROUND * math.sqrt(3 + (tiles + 1) / 2)
    A, B = values(kinds[0], 20_000 if way == "nt" else n, n if way == "nt" else 128, 3), values(kinds[1], 128 if way == "nt" else n, n if way == "nt" else 128, 4)
    got, want = (nt if way == "nt" else tn)(g, A, B)
    err = got - want
    assert rms(err) <= bound * rms(want)
    if kinds == ("uniform", "third") and way == "nt":
        # terms left out of the products of one weight would all have the same sign: 2e-8 on average for the three smallest but one
        assert abs(float((err / want).mean())) <= 4e-9


@pytest.mark.parametrize("kind", ["uniform", "normal"])
def test_many_rows(g, kind):
    """10^6 rows in 256 slices of 123 tiles, the slices added in 16 groups of 16.  n terms of one sign added in order: n roundings,
    in the mean square at 1/3 of the square of their sum; of random signs: at 1/2.  The errors of slices and of groups are independent,
    and a slice is 1/256 of the sum, or 1/16 of its size where signs are random."""
    A, B = values(kind, 1_000_000, 128, 5), values(kind, 1_000_000, 64, 6)
    got, want = tn(g, A, B)
    n = 123 / 3 / 256 + 16 / 3 / 16 + 16 / 3 if kind == "uniform" else 3 + 123 / 2 + 16 / 2 + 16 / 2
    assert rms(got - want) <= 1.25 * ROUND * math.sqrt(n) * rms(want)


@pytest.mark.parametrize("way,M,K,N", [("nt", 1_000_000, 256, 16), ("nt", 400_000, 32, 64), ("tn", 128, 1024, 1024), ("tn", 96, 1000, 1024)])
def test_errors_have_no_sign(g, way, M, K, N):
    """Column sums over many rows (bias gradients) add up the errors of the results: their mean has to vanish, to five times what the
    mean of that many independent errors has by chance, and 1/2000 of half a unit for the pairing of rows and tiles with opposite signs."""
    A, B = values("normal", M, K, 7), values("normal", *((N, K) if way == "nt" else (M, N)), 8)
    err, total = torch.zeros((), device=DEV, dtype=torch.float64), 0.0
    squares = torch.zeros((), device=DEV, dtype=torch.float64)
    if way == "nt":
        got = torch.empty(M, N, device=DEV)
        g.grp_gemm_nt(M, N, K, A, K, g.DTYPE_FP32, B, K, got, N)
        for lo in range(0, M, 100_000):
            want = A[lo:lo + 100_000].double() @ B.double().T
            e = got[lo:lo + 100_000].double() - want
            err, squares, total = err + e.sum(), squares + e.pow(2).sum(), total + float(want.pow(2).sum())
    else:
        got, want = tn(g, A, B)
        err, squares, total = (got - want).sum(), (got - want).pow(2).sum(), float(want.pow(2).sum())
    n = got.numel()
    size = math.sqrt(total / n)
    assert abs(float(err)) / n <= 5 * math.sqrt(float(squares) / n / n) + U / 2000 * size


@pytest.mark.parametrize("M,K,N", [(1, 65, 65), (33, 66, 96), (700, 128, 95), (5_000, 75, 130), (5_000, 130, 192), (3_000, 257, 161), (100_003, 75, 185), (31, 100, 288),
                                   (1, 65, 200), (33, 96, 100), (5_000, 66, 128), (700, 190, 256), (100_003, 81, 255), (3_000, 257, 97)])
@pytest.mark.parametrize("bf16,pad", [(False, 0), (False, 1), (True, 0)])
def test_tiles_of_96(g, M, K, N, bf16, pad):
    """Shapes whose tiles of 96 columns, or of 96 rows, leave less of them empty than tiles of 128, packed and with room at the rows' ends.  Every element is a
    sum in which at most M / 32 + 40 roundings follow one another (a k-tile's five, the tiles', the slices')."""
    A, B = values("normal", M, K, 11), values("normal", M, N, 12)
    if bf16:
        A = A.bfloat16()
    a, b = (torch.full((M, w + 7 * pad), float("nan"), device=DEV, dtype=t.dtype) for t, w in ((A, K), (B, N)))
    a[:, :K], b[:, :N] = A, B
    got = torch.full((K, N), float("nan"), device=DEV)
    ws = torch.empty(max(16, g.grp_gemm_tn_workspace_bytes(M, K, N)), dtype=torch.uint8, device=DEV)
    g.grp_gemm_tn(M, K, N, a, a.shape[1], g.DTYPE_BF16 if bf16 else g.DTYPE_FP32, b, b.shape[1], got, N, ws)
    want, size = A.double().T @ B.double(), A.double().abs().T @ B.double().abs()
    assert bool(((got.double() - want).abs() <= (M / 32 + 40) * U * size).all())
