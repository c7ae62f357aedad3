"""The counters that the parts of heavy items share in the per-vertex and
per-edge passes: they are there where pivots are heavy (the handle's memory
against a plan without parts), stay inside 64 MiB or 24 bytes an edge however
many pivots are, and every vertex and edge equals the oracle's."""

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


# pivots n_u, mids n_v, records drawn: 300 pivots of up to 1M wedges; 2,000 of
# up to 400K, most of them over the part budget, with windows of 128 KiB
@pytest.mark.parametrize("n_u,n_v,drawn", [(300, 30000, 2_800_000), (2000, 20000, 4_240_000)])
def test_room_of_heavy_items_counters(dbbc, n_u, n_v, drawn):
    rng = np.random.default_rng(n_u)
    key = np.unique(rng.integers(0, n_u * n_v, drawn))
    key = key[rng.permutation(len(key))]
    u, v = (key // n_v).astype(np.int32), (key % n_v).astype(np.int32)
    s = rng.choice([-1, 1], len(key)).astype(np.int8)
    r = vp_counts(n_u, n_v, u, v, s, per_vertex=True, per_edge=True)
    with dbbc.Graph(n_u, n_v, u, v, s) as h:
        held = []
        for flags in (0, dbbc.DBBC_OPT_HOST_PLAN):  # (the host planner cuts no items into parts)
            c, bu, bv, uu, uv = h.count_per_vertex(flags=flags)
            held.append(h.stats()["device_bytes"])
            assert (c.balanced, c.unbalanced, c.total) == (r.balanced, r.unbalanced, r.total)
            for t, want in ((bu, r.bal_u), (bv, r.bal_v), (uu, r.unb_u), (uv, r.unb_v)):
                assert np.array_equal(t.cpu().numpy(), want)
        counters = held[0] - held[1]
        lists = 1 << 20  # the parts' items, and groups packed otherwise
        assert counters > 8 << 20, "no item has parts"
        assert counters <= max(64 << 20, 24 * len(key)) + lists
        c, be, ue = h.count_per_edge()
        assert np.array_equal(be.cpu().numpy(), r.bal_e) and np.array_equal(ue.cpu().numpy(), r.unb_e)
