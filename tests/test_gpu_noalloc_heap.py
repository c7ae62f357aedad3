"""dbbc_count_noalloc asks for no heap memory, with and without a dense block (a
process of its own counts the library's calls of operator new), and launches
with more buffers to clear than one clearing launch takes."""

import os
import subprocess
import sys

import pytest

from oracle import vp_counts
from synth import chung_lu_graph

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = r"""
import ctypes, sys
counter = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
counter.new_count.restype = ctypes.c_long
sys.path.insert(0, sys.argv[2])
import torch
import paper_2609_21848_amd as dbbc
from synth import chung_lu_graph
torch.cuda.set_device(0)
g = chung_lu_graph(6000, 5000, 120000, 2.1, 1.9, 0.4, seed=31)
lib = dbbc.load()
counter.new_watch(ctypes.cast(lib.dbbc_count_noalloc, ctypes.c_void_p))
with dbbc.Graph(g.n_u, g.n_v, g.u, g.v, g.sign) as h:
    assert counter.new_count() > 0, "the library's calls are not counted"
    for opts in ({}, dict(hub_T=256, window_L=1024), dict(part_work=4096, hub_T=128)):
        want = tuple(h.count(**opts))
        o, c = dbbc.Options(**opts), dbbc._Counts()
        for _ in range(3):
            before = counter.new_count()
            rc = lib.dbbc_count_noalloc(h.handle, ctypes.byref(o), ctypes.byref(c), None)
            made = counter.new_count() - before
            assert rc == 0 and (c.balanced, c.unbalanced, c.total, c.wedges) == want, (opts, rc)
            print("blocks", opts, made, flush=True)
            assert made == 0, (opts, made)
"""


@pytest.fixture(scope="module")
def dbbc():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    import paper_2609_21848_amd as mod
    mod.load()
    return mod


def test_noalloc_makes_no_heap_block(dbbc, tmp_path):
    so = str(tmp_path / "new_count.so")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-o", so,
                           os.path.join(ROOT, "tests", "native", "new_count.cpp"), "-ldl"])
    r = subprocess.run([sys.executable, "-c", CHILD, so, ROOT], capture_output=True, text=True, timeout=110)
    assert r.returncode == 0, r.stdout + r.stderr
    assert r.stdout.count("blocks") == 9


# two planes to clear per graph with a dense block, and the control words and
# the results: 10, 12, 14 and 26 ranges
@pytest.mark.parametrize("k", [4, 5, 6, 12])
@pytest.mark.parametrize("capture", [False, True])
def test_batches_around_the_ranges_of_one_launch(dbbc, k, capture):
    gs = [chung_lu_graph(400 + 10 * i, 300 + 7 * i, 6000, 2.1, 1.9, 0.4, seed=i) for i in range(k)]
    want = [vp_counts(g.n_u, g.n_v, g.u, g.v, g.sign) for g in gs]
    hs = [dbbc.Graph(g.n_u, g.n_v, g.u, g.v, g.sign) for g in gs]
    with dbbc.Batch(hs, capture=capture, hub_T=128) as b:
        for _ in range(3):  # every launch starts from zero
            for got, r in zip(b.count(), want):
                assert tuple(got) == (r.balanced, r.unbalanced, r.total, r.wedges)
    for h in hs:
        h.close()
