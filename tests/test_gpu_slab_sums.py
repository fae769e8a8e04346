"""Neighbour sums in slabs of columns (many rows, or long rows with the sliced schedule) against sums in float64 over every width class: part
vectors, part slabs, several slabs, pitches that keep them to the general kernel, rows that end anywhere, row counts around the rule's."""
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu
DEV = "cuda"
MANY = 1 << 17


def _check(g, part, src, dst, n, F, dtype, pitch, offset=0):
    print(f"[case] slab sums n={n} F={F} {dtype} pitch={pitch}", flush=True)
    buf = torch.full((n, pitch), float("nan"), device=DEV, dtype=dtype)
    x = buf[:, offset:offset + F]
    x.copy_(torch.randn(n, F, generator=torch.Generator(device=DEV).manual_seed(F), device=DEV))
    if pitch - offset >= (F + 3) // 4 * 4 > F:
        buf[:, offset + F:offset + (F + 3) // 4 * 4] = 0       # the pad columns of a row's last vector
    x[7] = float("inf")
    for transposed, self_term, scale in ((False, True, g.SCALE_MEAN), (True, False, g.SCALE_NONE)):
        to, frm = (src, dst) if transposed else (dst, src)
        deg = torch.bincount(to, minlength=n).double()
        want, size = torch.zeros(n, F, dtype=torch.float64, device=DEV), torch.zeros(n, F, dtype=torch.float64, device=DEV)
        xd = x.double()
        want.index_add_(0, to, xd[frm])
        size.index_add_(0, to, xd[frm].abs())
        if self_term:
            want += xd
            size += xd.abs()
        a = 1 / deg.clamp(min=1) if scale == g.SCALE_MEAN else torch.ones_like(deg)
        ldy = (F + 3) // 4 * 4 + 4                             # (up to a multiple of four the columns are padding)
        y = torch.full((n, ldy), float("nan"), device=DEV)
        g.grp_spmm(part, transposed, scale, self_term, F, x, pitch, g.DTYPE_BF16 if dtype == torch.bfloat16 else g.DTYPE_FP32, y[:, :F], ldy)
        torch.cuda.synchronize()
        inf = torch.isinf(want).any(1)
        assert torch.isinf(y[:, :F][inf]).all()
        # a sum of k terms added in any order is off by at most (k + 1) roundings of its terms' magnitude (deg + self + scale)
        bound = (size * a[:, None]) * ((deg[:, None] + 3) * 2.0 ** -24)
        err = (y[:, :F].double() - want * a[:, None]).abs()
        assert (err[~inf] <= bound[~inf] + 1e-30).all()
        assert torch.isnan(y[:, ldy - 4:]).all()


WIDTHS = [(torch.float32, f, p, o) for f, p, o in ((9, 12, 0), (16, 16, 0), (17, 20, 0), (31, 36, 4), (33, 36, 0), (64, 64, 0), (64, 68, 4),
                                                    (96, 96, 0), (100, 100, 0), (128, 160, 32), (176, 192, 0), (200, 224, 0), (1000, 1024, 0))]
WIDTHS += [(torch.bfloat16, f, p, o) for f, p, o in ((32, 32, 0), (24, 40, 8), (64, 64, 0), (72, 72, 0), (128, 128, 0), (200, 256, 0), (256, 256, 0), (130, 132, 0))]


@pytest.fixture(scope="module")
def lib():
    import paper_2602_01872_amd as g
    g.load()
    return g


@pytest.mark.parametrize("n,E,sliced", [(MANY - 1, 300_000, False), (MANY, 1_500_000, False), (MANY + 259, 2_000_000, True), (3000, 200_000, True)])
def test_sums(lib, n, E, sliced):
    g = lib
    src, dst = (t.to(DEV) for t in synth.rmat_graph(max(2, (n - 1).bit_length()), E, seed=n, n_nodes=n))
    if sliced:
        g.grp_set_slice_policy(1, 1)
    try:
        part = g.grp_partition_from_local_coo(src, dst, n)
    finally:
        g.grp_set_slice_policy()
    for dtype, F, pitch, offset in WIDTHS:
        if n * F <= 150 << 20:
            _check(g, part, src, dst, n, F, dtype, pitch, offset)
    part.destroy()


def test_rows_longer_than_any_bin_without_a_split(lib):
    """A structure whose only long row is below the split, rows of no edges at both ends, and a last row that ends with the indices."""
    g = lib
    n = MANY + 5
    deg = torch.zeros(n, dtype=torch.int64)
    deg[3], deg[n // 2], deg[n - 1] = 128, 127, 1
    dst = torch.repeat_interleave(torch.arange(n), deg)
    src = torch.arange(dst.numel()) * 37 % n
    part = g.grp_partition_from_local_coo(src.to(DEV), dst.to(DEV), n)
    _check(g, part, src.to(DEV), dst.to(DEV), n, 64, torch.float32, 64)
    _check(g, part, src.to(DEV), dst.to(DEV), n, 16, torch.float32, 16)


@pytest.mark.parametrize("n", [1 << 22, (1 << 22) + 1])
def test_operand_of_four_gib(lib, n):
    """X of exactly 4 GiB, the most that 32-bit offsets from a slab's first column reach, and of one row more; the last rows are
    neighbours of short rows and of a long one, whose edges go by the sliced schedule."""
    g = lib
    gen = torch.Generator().manual_seed(n)
    src = torch.cat([torch.randint(n, (200_000,), generator=gen), torch.arange(n - 4000, n), torch.arange(n - 64, n)])
    dst = torch.cat([torch.randint(n, (200_000,), generator=gen), torch.full((4000,), 5), torch.arange(n - 64, n).flip(0)])
    src, dst = src.to(DEV), dst.to(DEV)
    g.grp_set_slice_policy(1, 1)
    try:
        part = g.grp_partition_from_local_coo(src, dst, n)
    finally:
        g.grp_set_slice_policy()
    _check(g, part, src, dst, n, 256, torch.float32, 256)
    part.destroy()
    torch.cuda.empty_cache()


@pytest.mark.parametrize("n", [1 << 22, (1 << 22) + 1])
def test_short_rows_over_an_operand_of_four_gib(lib, n):
    """The same sizes with rows so unequal (a long row of a tenth of the edges) that the short ones go by slabs, and by the general kernel a
    row above."""
    g = lib
    gen = torch.Generator().manual_seed(n)
    src = torch.cat([torch.randint(n, (100_000,), generator=gen), torch.arange(n - 12_000, n), torch.arange(n - 64, n)])
    dst = torch.cat([torch.randint(n, (100_000,), generator=gen), torch.full((12_000,), 5), torch.arange(n - 64, n).flip(0)])
    src, dst = src.to(DEV), dst.to(DEV)
    part = g.grp_partition_from_local_coo(src, dst, n)
    _check(g, part, src, dst, n, 256, torch.float32, 256)
    part.destroy()
    torch.cuda.empty_cache()


@pytest.mark.parametrize("deg", [0, 3, 6, 31, 32])
def test_rows_of_like_lengths(lib, deg):
    """Both sides of the rule that leaves short rows of like lengths to the general kernel, and rows that are all empty but one."""
    g = lib
    n = MANY + 3
    gen = torch.Generator().manual_seed(deg)
    dst = torch.arange(n).repeat_interleave(deg) if deg else torch.full((9,), n - 1)
    src = torch.randint(n, (dst.numel(),), generator=gen)
    src, dst = src.to(DEV), dst.to(DEV)
    part = g.grp_partition_from_local_coo(src, dst, n)
    for dtype, F in ((torch.float32, 16), (torch.float32, 64), (torch.float32, 128), (torch.bfloat16, 32), (torch.bfloat16, 64)):
        _check(g, part, src, dst, n, F, dtype, F)
    part.destroy()


@pytest.mark.parametrize("F,bf16", [(16, False), (32, False), (32, True), (64, True)])
def test_sums_are_as_accurate_as_four_chains(F, bf16):
    """Narrow rows of 100 edges: the rounding errors are those of chains of a quarter of a row at most (one chain has 1.8 to 3 times as much)."""
    import paper_2602_01872_amd as g
    print(f"[case] accuracy of slab sums F={F} bf16={bf16}", flush=True)
    n, deg = 1 << 17, 100
    gen = torch.Generator(device=DEV).manual_seed(F)
    s, d = torch.randint(n, (n * deg,), generator=gen, device=DEV), torch.arange(n, device=DEV).repeat_interleave(deg)
    part = g.grp_partition_from_local_coo(s, d, n)
    col = torch.from_numpy(part.array("col")).to(DEV).long().view(n, deg)
    for x in (torch.randn(n, F, generator=gen, device=DEV), torch.rand(n, F, generator=gen, device=DEV) + 0.1):
        x = x.to(torch.bfloat16) if bf16 else x
        y, want, chain = torch.empty(n, F, device=DEV), torch.zeros(n, F, dtype=torch.float64, device=DEV), torch.zeros(4, n, F, device=DEV)
        g.grp_spmm(part, False, g.SCALE_NONE, False, F, x, F, g.DTYPE_BF16 if bf16 else g.DTYPE_FP32, y, F)
        for e in range(deg):
            want += x[col[:, e]].double()
            chain[e % 4] += x[col[:, e]].float()
        four = (chain[0] + chain[1]) + (chain[2] + chain[3])
        assert float((y - want).norm()) <= 1.1 * float((four - want).norm())
