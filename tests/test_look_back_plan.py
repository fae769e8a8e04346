"""The prefix sums of a sampled step wait for each other's workgroups within a launch: however many layers and merged steps share it, few
enough of them wait that launches on several streams cannot keep each other from the GPU (CPU only: the plan alone is called)."""
import ctypes as C
import os

import pytest

WAITING = 384                                                # a launch's workgroups that may wait


class Plan(C.Structure):
    _fields_ = [("rounds", C.c_int), ("parts", C.c_int)]


@pytest.mark.parametrize("steps", [1, 2, 4, 7, 8])
@pytest.mark.parametrize("layers", [1, 2, 3, 7, 15])
def test_waiting_workgroups_of_a_launch(steps, layers):
    import paper_2602_01872_amd as g
    if not os.path.exists(g.LIB_PATH):
        import __graft_entry__
        __graft_entry__.build()
    fn = getattr(g.load(), "_ZN3grp14look_back_planElli")    # ScanPlan grp::look_back_plan(items, round, sums)
    fn.argtypes, fn.restype = [C.c_int64, C.c_int64, C.c_int], Plan
    for round_ in (1024, 4096):
        for items in (1, 2, 1023, 1024, 1025, 70_001, 1 << 20, (1 << 20) + 1, 7_000_000, (1 << 31) - 1):
            p = fn(items, round_, steps * layers)
            assert 1 <= p.parts <= 128 and p.parts * steps * layers <= WAITING
            assert p.parts * p.rounds * round_ >= items > (p.parts - 1) * p.rounds * round_
