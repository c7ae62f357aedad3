"""The workgroups of a direct launch (CPU): the rule picks the shape that was the
faster one, by 5 % or more, in launches timed with both on 256 CUs, and never a
narrow workgroup for windows that its counters do not hold."""

import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def narrow(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("shape") / "direct_shape.so")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-o", so,
                           os.path.join(ROOT, "tests", "native", "direct_shape.cpp")])
    f = ctypes.CDLL(so).direct_is_narrow
    f.argtypes = [ctypes.c_int, ctypes.c_uint64, ctypes.c_uint64, ctypes.c_int, ctypes.c_int]
    return lambda *a: bool(f(*a))


# items, wedges, heaviest item, widest window; wide and narrow us
@pytest.mark.parametrize("n,w,heaviest,keys,wide_us,narrow_us", [
    (672, 224250000, 437988, 5000, 148.5, 186.5),      # few heavy pivots in parts
    (614, 159200000, 310937, 8000, 136.0, 151.3),
    (921, 1467900000, 2866992, 6000, 858.9, 982.4),    # (its runs all staged)
    (66, 9800000, 262144, 8000, 54.4, 83.6),
    (1343, 27323090, 262144, 8000, 41.1, 61.8),        # skewed graphs: one item outlasts the rest
    (909, 10531719, 225204, 16000, 41.5, 64.0),
    (328, 2530528, 75742, 8000, 20.6, 27.8),
    (843, 9654698, 35467, 500, 21.4, 23.5),
    (1991, 161732126, 182105, 8000, 119.7, 107.9),     # many like items
    (3987, 373614330, 214549, 8000, 223.8, 197.9),
    (2999, 12959153376, 7949448, 3000, 3492.0, 3237.0),
    (16262, 3998000000, 262144, 2000, 1380.8, 1236.5),
    (25406, 65663330, 25953, 3997, 582.7, 497.6),      # batches
    (4692, 14681034, 34674, 2987, 155.1, 135.8),
    (13269, 81364905, 109825, 14977, 395.9, 338.9),
    (1231, 10042525, 173329, 6257, 93.9, 115.6),
    (7632, 71684126, 204931, 7337, 239.9, 257.1),
])
def test_the_faster_shape_is_picked(narrow, n, w, heaviest, keys, wide_us, narrow_us):
    assert narrow(n, w, heaviest, keys, 256) == (narrow_us < wide_us)


@pytest.mark.parametrize("keys", [16385, 20000, 32768])
def test_wide_windows_take_wide_workgroups(narrow, keys):
    assert narrow(25406, 65663330, 25953, 16384, 256)
    assert not narrow(25406, 65663330, 25953, keys, 256)
