"""The rule by which several groups of lanes share a row of a neighbour sum never takes a launch past the 2^32 work-items that one may
hold, whatever the rows and the chunks of split rows beside them (CPU only: the rule alone is called)."""
import ctypes as C
import os

import pytest


@pytest.fixture(scope="module")
def share():
    import paper_2602_01872_amd as g
    if not os.path.exists(g.LIB_PATH):
        import __graft_entry__
        __graft_entry__.build()
    fn = getattr(g.load(), "_ZN3grp10spmm_shareElllii")      # bool grp::spmm_share(rows, edges, chunks, G, S)
    fn.argtypes = [C.c_int64, C.c_int64, C.c_int64, C.c_int, C.c_int]
    fn.restype = C.c_bool
    return fn


@pytest.mark.parametrize("G", [1, 2, 4, 8, 16, 32])
def test_shared_rows_fit_a_launch(share, G):
    S = 2 if G == 32 else 4
    per_group = 256 // (G * S)                               # rows of a workgroup
    limit = 1 << 24                                          # workgroups of a launch, not reached
    for chunks in (0, 1, 4_200_000, (1 << 22) + 1, 9_000_000, limit - 2):
        room = limit - 1 - chunks                            # workgroups left for the rows
        for rows in (1, room * per_group - 1, room * per_group, room * per_group + 1, 100_000_000, (1 << 31) - 1):
            fits = chunks + -(-rows // per_group) < limit
            for degree in (1, 3, 8, 40):
                if share(rows, rows * degree, chunks, G, S):
                    assert fits, (rows, degree, chunks)
            if G <= 2:                                       # narrow rows share whenever the launch can hold them
                assert share(rows, rows, chunks, G, S) == fits
