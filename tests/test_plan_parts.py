"""The direct items of a count plan (CPU): heaviest first, the parts of split
pivots among the pivots that are whole; and the part budget raised, in the one
plan, until the parts' counters fit their room."""

import ctypes
import os
import subprocess

import numpy as np
import pytest

from synth import chung_lu_graph

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("parts") / "plan_parts.so")
    native = os.path.join(ROOT, "tests", "native")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-o", so,
                           os.path.join(native, "plan_parts.cpp"), os.path.join(native, "host_build.cpp"),
                           os.path.join(ROOT, "paper_2609_21848_amd", "csrc", "plan.cpp")])
    return ctypes.CDLL(so)


@pytest.mark.parametrize("part_work", [4096, 20000, 1 << 24])
def test_parts_are_ordered_with_the_others(lib, part_work):
    g = chung_lu_graph(3000, 2000, 60000, 2.0, 1.9, 0.4, seed=5)
    out = np.zeros(4, np.int64)
    i32, i64, p = ctypes.c_int32, ctypes.c_int64, ctypes.c_void_p
    lib.plan_parts.argtypes = [i32, i32, i64, p, p, p, i32, p]
    assert lib.plan_parts(g.n_u, g.n_v, g.m, g.u.ctypes.data, g.v.ctypes.data, g.sign.ctypes.data, part_work,
                          out.ctypes.data) == 0
    ordered, parts, whole, before_last = out
    assert ordered
    if part_work < 1 << 24:
        assert parts > 0 and 0 < before_last <= whole
    else:
        assert parts == 0 and whole > 0


def test_parts_fit_their_room(lib):
    g = chung_lu_graph(3000, 2000, 60000, 2.0, 1.9, 0.4, seed=5)
    i32, i64, p = ctypes.c_int32, ctypes.c_int64, ctypes.c_void_p
    lib.plan_room.argtypes = [i32, i32, i64, p, p, p, i32, i64, p]

    def plan(room):
        out = np.zeros(4, np.int64)
        assert lib.plan_room(g.n_u, g.n_v, g.m, g.u.ctypes.data, g.v.ctypes.data, g.sign.ctypes.data, 4096, room,
                             out.ctypes.data) == 0
        return out.tolist()
    free, parts, wedges, reduces = plan(1 << 40)
    assert parts > 100 and reduces > 0
    seen = {parts}
    for room in (free, free - 1, free // 5, free // 50, 1):
        held, parts, w, reduces = plan(room)
        assert held <= room or parts == 0  # (the reverse items' parts keep theirs)
        assert w == wedges and (parts == 0) == (reduces == 0)
        seen.add(parts)
    assert len(seen) > 2 and 0 in seen
