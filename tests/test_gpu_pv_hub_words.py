"""Per-vertex and per-edge passes on hub pivots whose pairs' completed counts
take the place of the item's own counter words, below 2^16 wedges and with one
pair at the bound or past it (that item reads them from the dense block's planes).
Every vertex's and edge's counts (integers) must equal the oracle's."""

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


@pytest.mark.parametrize("common", [3000, 65535, 65536, 70000])
@pytest.mark.parametrize("hub_T", [0, 128])
def test_hub_pairs_around_two_bytes(dbbc, common, hub_T):
    rng = np.random.default_rng(common + hub_T)
    n_u, n_v = common + 500, 700
    u = [np.tile(np.arange(common), 2), rng.integers(0, n_u, 60000)]
    v = [np.repeat([3, 5], common), rng.integers(6, n_v, 60000)]
    key = np.unique(np.concatenate(u).astype(np.int64) * n_v + np.concatenate(v))
    key = key[rng.permutation(len(key))]
    u, v = (key // n_v).astype(np.int32), (key % n_v).astype(np.int32)
    s = rng.choice([-1, 1], len(key), p=[0.1, 0.9]).astype(np.int8)
    r = vp_counts(n_u, n_v, u, v, s, per_vertex=True, per_edge=True)
    with dbbc.Graph(n_u, n_v, u, v, s) as h:
        c, bu, bv, uu, uv = h.count_per_vertex(hub_T=hub_T)
        assert (c.balanced, c.unbalanced, c.total) == (r.balanced, r.unbalanced, r.total)
        for t, want in ((bu, r.bal_u), (bv, r.bal_v), (uu, r.unb_u), (uv, r.unb_v)):
            assert np.array_equal(t.cpu().numpy(), want)
        for flags in (0, dbbc.DBBC_OPT_WIDE_EDGES):
            c, be, ue = h.count_per_edge(flags=flags, hub_T=hub_T)
            assert np.array_equal(be.cpu().numpy(), r.bal_e) and np.array_equal(ue.cpu().numpy(), r.unb_e)
