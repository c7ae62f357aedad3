"""Per-vertex and per-edge passes on graphs whose heaviest direct items are cut
into parts that share their counters: several parts per item on both sides,
with and without a dense block, key windows around the keys a sweep step takes,
and an item of more than 2^16 runs (its counters take 32 bits each, in two
windows).
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


def _heavy(n_u, n_v, hubs, hub_deg, mids_deg, seed):
    """A few hubs on either side over vertices of moderate degree."""
    rng = np.random.default_rng(seed)
    u = [rng.integers(0, n_u, mids_deg * n_v), np.repeat(np.arange(hubs), hub_deg),
         rng.integers(0, n_u, hubs * hub_deg // 4)]
    v = [np.repeat(np.arange(n_v), mids_deg), rng.integers(0, n_v, hubs * hub_deg),
         np.repeat(n_v - 1 - np.arange(hubs), hub_deg // 4)]
    key = np.unique(np.concatenate(u).astype(np.int64) * n_v + np.concatenate(v))
    key = key[rng.permutation(len(key))]
    return ((key // n_v).astype(np.int32), (key % n_v).astype(np.int32),
            rng.choice([-1, 1], len(key)).astype(np.int8))


@pytest.mark.parametrize("n_u,n_v,hubs,hub_deg,mids_deg", [
    (1023, 5000, 6, 4500, 24), (4097, 9000, 3, 8000, 30), (33000, 12000, 5, 11000, 26), (2500, 2600, 40, 2000, 60),
    (18001, 70000, 2, 68000, 4)])
@pytest.mark.parametrize("opts", [{}, dict(hub_T=512), dict(window_L=1024, reverse_L=256, hub_T=0)])
def test_parts_of_heavy_items(dbbc, n_u, n_v, hubs, hub_deg, mids_deg, opts):
    u, v, s = _heavy(n_u, n_v, hubs, hub_deg, mids_deg, n_u)
    r = vp_counts(n_u, n_v, u, v, s, per_vertex=True, per_edge=True)
    with dbbc.Graph(n_u, n_v, u, v, s) as h:
        for _ in range(2):  # the accumulators start at zero again
            c, bu, bv, uu, uv = h.count_per_vertex(**opts)
            assert (c.balanced, c.unbalanced, c.total) == (r.balanced, r.unbalanced, r.total)
            for t, want in ((bu, r.bal_u), (bv, r.bal_v), (uu, r.unb_u), (uv, r.unb_v)):
                assert np.array_equal(t.cpu().numpy(), want)
            for flags in (0, dbbc.DBBC_OPT_WIDE_EDGES):
                c, be, ue = h.count_per_edge(flags=flags, **opts)
                assert np.array_equal(be.cpu().numpy(), r.bal_e) and np.array_equal(ue.cpu().numpy(), r.unb_e)
