"""Which builds are sorted by buckets: every one of at most 2^22 nodes and 2^26 edges, with keys that fit 32 bits and at most 4096 buckets of
each direction (CPU only: the plan alone is called)."""
import ctypes as C
import os

import pytest


class Plan(C.Structure):
    _fields_ = [("row_bits", C.c_int), ("id_bits", C.c_int), ("n_buckets", C.c_int)]


@pytest.fixture(scope="module")
def plan():
    import paper_2602_01872_amd as g
    if not os.path.exists(g.LIB_PATH):
        import __graft_entry__
        __graft_entry__.build()
    fn = getattr(g.load(), "_ZN3grp11bucket_planEllPNS_10BucketPlanE")       # bool grp::bucket_plan(n, nnz, plan)
    fn.argtypes, fn.restype = [C.c_int64, C.c_int64, C.c_void_p], C.c_bool
    return fn


@pytest.mark.parametrize("nnz", [1, 5000, 1 << 20, 5_000_000, 9_000_000, 1 << 24, 1 << 26])
def test_every_build_within_the_limits(plan, nnz):
    for n in (1, 2, 3, 2047, 2048, 2049, 70_001, 1 << 20, (1 << 21) - 1, 1 << 21, (1 << 21) + 1, 3_000_000, (1 << 22) - 1, 1 << 22):
        p = Plan()
        assert plan(n, nnz, C.addressof(p)), n
        assert (1 << p.id_bits) >= n and p.row_bits + p.id_bits <= 32 and 0 <= p.row_bits <= 11
        assert (p.n_buckets - 1) << p.row_bits < n <= p.n_buckets << p.row_bits and p.n_buckets <= 4096
    p = Plan()
    assert not plan((1 << 22) + 1, nnz, C.addressof(p)) and not plan(5, (1 << 26) + 1, C.addressof(p)) and not plan(0, 0, C.addressof(p))
