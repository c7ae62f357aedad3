"""dbbc_count_noalloc beside a dense block that the caller sizes: the parts of
heavy pivots take what the block's planes leave of the scratch, so every block
that fits by itself is counted, with the results of the oracle."""

import ctypes

import numpy as np
import pytest

from oracle import vp_counts

pytestmark = pytest.mark.gpu


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
def heavy():
    # 300 pivots of 2^18 to 2^20 wedges each over 30,000 vertices: several
    # parts a pivot by default, a window of 30,000 counters each
    n_u, n_v = 300, 30000
    rng = np.random.default_rng(17)
    key = np.unique(rng.integers(0, n_u * n_v, 2_800_000))
    key = key[rng.permutation(len(key))]
    u, v = (key // n_v).astype(np.int32), (key % n_v).astype(np.int32)
    s = rng.choice([-1, 1], len(key)).astype(np.int8)
    return n_u, n_v, u, v, s, vp_counts(n_u, n_v, u, v, s)


@pytest.mark.parametrize("hub_T,parts", [(0, True), (128, True), (1024, None), (1920, None), (2560, None)])
def test_parts_leave_the_block_its_room(dbbc, heavy, hub_T, parts):
    n_u, n_v, u, v, s, r = heavy
    want = (r.balanced, r.unbalanced, r.total, r.wedges)
    with dbbc.Graph(n_u, n_v, u, v, s) as h:
        assert tuple(h.count(hub_T=hub_T, flags=dbbc.DBBC_OPT_TIME_KERNELS)) == want
        reduces = sum(k["items"] for k in h.kernel_times() if k["name"] == "reduce")
        if parts:
            assert reduces > 0, "no pivot has parts"
        lib, c, o = dbbc.load(), dbbc._Counts(), dbbc.Options(hub_T=hub_T)
        h.count(hub_T=hub_T)
        rc = lib.dbbc_count_noalloc(h.handle, ctypes.byref(o), ctypes.byref(c), None)
        assert rc == 0, lib.dbbc_last_error()
        assert (c.balanced, c.unbalanced, c.total, c.wedges) == want
