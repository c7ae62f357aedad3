"""The device graph build at the sizes where its sorts change shape: one tile
and the next, the switch between tile sizes, one to four digits per key,
records dropped across that switch, and rows whose wedges take a whole
wavefront to decide.  Counts by record (they go through every array of the
build) against the oracle; all values are integers and must be equal."""

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


def _active(n_u, n_v, u, v):
    """Pivots with a wedge: some lower-priority neighbour has a neighbour of
    lower priority than the pivot (priority: degree, then global id)."""
    a = np.concatenate([u, v + n_u])
    b = np.concatenate([v + n_u, u])
    deg = np.bincount(a, minlength=n_u + n_v)
    prio = deg.astype(np.int64) * (n_u + n_v) + np.arange(n_u + n_v)
    low = np.full(n_u + n_v, np.iinfo(np.int64).max)
    np.minimum.at(low, b, prio[a])  # the lowest neighbour of every mid
    return len(np.unique(a[(prio[b] < prio[a]) & (low[b] < prio[a])]))


def _check(dbbc, n_u, n_v, u, v, s):
    key = u.astype(np.int64) * n_v + v
    last = np.sort(len(u) - 1 - np.unique(key[::-1], return_index=True)[1])  # the record kept of each pair
    r = vp_counts(n_u, n_v, u[last], v[last], s[last], per_edge=True)
    with dbbc.Graph(n_u, n_v, u, v, s) as h:
        st = h.stats()
        c, be, ue = h.count_per_edge()
        assert tuple(h.count()) == (r.balanced, r.unbalanced, r.total, r.wedges)
    assert (c.balanced, c.unbalanced) == (r.balanced, r.unbalanced)
    assert (st["m"], st["dups_dropped"], st["wedges_vp"]) == (len(last), len(u) - len(last), r.wedges)
    assert st["pivots_active"] == _active(n_u, n_v, u[last].astype(np.int64), v[last].astype(np.int64))
    for got, want in ((be, r.bal_e), (ue, r.unb_e)):
        full = np.zeros(len(u), np.int64)
        full[last] = want
        assert np.array_equal(got.cpu().numpy(), full)


@pytest.mark.parametrize("m,n_u,n_v", [
    (1, 1, 1), (2, 1, 2), (255, 40, 16), (1023, 300, 255), (1024, 256, 257), (1025, 300, 256), (4097, 2049, 100),
    (20000, 65536, 65537), (70000, 70001, 300), (30000, 17_000_000, 40)])
def test_record_and_vertex_counts_at_tile_edges(dbbc, m, n_u, n_v):
    rng = np.random.default_rng(m)
    u = rng.integers(0, n_u, m).astype(np.int32)
    v = rng.integers(0, n_v, m).astype(np.int32)
    u[0], v[-1] = n_u - 1, n_v - 1
    _check(dbbc, n_u, n_v, u, v, rng.choice([-1, 1], m).astype(np.int8))


@pytest.mark.parametrize("m,repeats", [((1 << 20) - 1, 0), (1 << 20, 0), ((1 << 20) + 1, 5), ((1 << 20) + 4096, 60000)])
def test_switch_of_tile_size_and_records_dropped_across_it(dbbc, m, repeats):
    rng = np.random.default_rng(m + repeats)
    n_u, n_v = 150_000, 90_000
    key = rng.choice(n_u * n_v, m - repeats, replace=False)
    key = np.concatenate([rng.choice(key, repeats), key])[rng.permutation(m)]
    _check(dbbc, n_u, n_v, (key // n_v).astype(np.int32), (key % n_v).astype(np.int32),
           rng.choice([-1, 1], m).astype(np.int8))


@pytest.mark.parametrize("a,b", [(1, 300), (300, 1), (30, 200), (200, 30), (129, 129)])
def test_complete_graphs_and_stars(dbbc, a, b):
    u, v = (x.ravel().astype(np.int32) for x in np.meshgrid(np.arange(a), np.arange(b), indexing="ij"))
    rng = np.random.default_rng(a)
    p = rng.permutation(a * b)
    _check(dbbc, a + 3, b + 2, u[p], v[p], rng.choice([-1, 1], a * b).astype(np.int8))
