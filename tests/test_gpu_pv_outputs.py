"""Where the per-vertex outputs lie: inside an allocation, at its very end, off
the word grid, and in host memory they are written; an allocation that ends
before the output does is refused, as the copies to it always were."""

import ctypes

import numpy as np
import pytest

from oracle import vp_counts
from synth import uniform_graph

pytestmark = pytest.mark.gpu

N_U, N_V = 60, 50  # a few hundred bytes an output: all inside one page


@pytest.fixture(scope="module")
def dbbc():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    import paper_2609_21848_amd as mod
    mod.load()
    return mod


@pytest.fixture(scope="module")
def hip(dbbc):
    lib = ctypes.CDLL("libamdhip64.so.7")  # the runtime that is loaded already
    lib.hipMalloc.argtypes = [ctypes.POINTER(ctypes.c_void_p), ctypes.c_size_t]
    lib.hipMemcpy.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_int]
    lib.hipFree.argtypes = [ctypes.c_void_p]
    return lib


class Block:
    """A hipMalloc of exactly `size` bytes, zeroed."""

    def __init__(self, hip, size):
        self.hip, self.size, p = hip, size, ctypes.c_void_p()
        assert hip.hipMalloc(ctypes.byref(p), size) == 0
        self.p = p.value
        zero = np.zeros(size, np.uint8)
        assert hip.hipMemcpy(self.p, zero.ctypes.data, size, 1) == 0

    def read(self):
        out = np.empty(self.size, np.uint8)
        assert self.hip.hipMemcpy(out.ctypes.data, self.p, self.size, 2) == 0
        return out

    def __enter__(self):
        return self

    def __exit__(self, *exc):
        self.hip.hipFree(self.p)


def _graph():
    g = uniform_graph(N_U, N_V, 900, 0.4, seed=3)
    return g, vp_counts(g.n_u, g.n_v, g.u, g.v, g.sign, per_vertex=True)


@pytest.mark.parametrize("before,after", [(0, 0), (8, 0), (0, 24), (4, 0), (1, 7)])
def test_outputs_anywhere_in_an_allocation(dbbc, hip, before, after):
    g, r = _graph()
    with dbbc.Graph(g.n_u, g.n_v, g.u, g.v, g.sign) as h, Block(hip, before + 8 * N_U + after) as b:
        assert dbbc.load().dbbc_count_per_vertex(h.handle, None, b.p + before, None, None, None, None, None) == 0
        got = b.read()
        assert np.array_equal(got[before:before + 8 * N_U].copy().view(np.int64), r.bal_u)
        assert not got[:before].any() and not got[before + 8 * N_U:].any()


@pytest.mark.parametrize("short", [1, 8, 8 * (N_U - 1)])
@pytest.mark.parametrize("offset", [0, 16])
def test_allocation_too_small_is_refused(dbbc, hip, short, offset):
    g, r = _graph()
    with dbbc.Graph(g.n_u, g.n_v, g.u, g.v, g.sign) as h, Block(hip, offset + 8 * N_U - short) as b:
        rc = dbbc.load().dbbc_count_per_vertex(h.handle, None, b.p + offset, None, None, None, None, None)
        assert rc == -6, rc  # DBBC_E_DEVICE
        assert not b.read().any()
        # the handle goes on
        c, bu, *_ = h.count_per_vertex()
        assert np.array_equal(bu.cpu().numpy(), r.bal_u)
