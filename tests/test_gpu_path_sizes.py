"""The inputs of the tests of small-group teams and of unpacked items' parts take
the paths that those tests are about: groups on either side of five a CU, and
an item of more than 2^16 runs whose two key windows are cut into parts."""

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


def test_groups_on_both_sides_of_the_team_bound(dbbc):
    import torch
    bound = 5 * torch.cuda.get_device_properties(0).multi_processor_count
    groups = []
    for m, n in ((300, 20), (30000, 9000), (170000, 50000), (260000, 50000), (400000, 50000)):
        rng = np.random.default_rng(m)
        key = np.unique(rng.integers(0, n * n, m))
        key = key[rng.permutation(len(key))]
        u, v = (key // n).astype(np.int32), (key % n).astype(np.int32)
        s = rng.choice([-1, 1], len(key)).astype(np.int8)
        with dbbc.Graph(n, n, u, v, s) as h:
            h.count(flags=dbbc.DBBC_OPT_TIME_KERNELS)
            groups += [k["items"] for k in h.kernel_times() if k["name"] == "small"]
    assert sum(0 < g <= bound for g in groups) >= 2, (groups, bound)
    assert sum(g > bound for g in groups) >= 1, (groups, bound)


def _wide_hubs(n_u, n_v, hubs, deg, seed):
    """Hubs of exactly deg neighbours each over vertices of degree 4."""
    rng = np.random.default_rng(seed)
    u = [rng.integers(hubs, n_u, 4 * n_v)] + [np.full(deg, h) for h in range(hubs)]
    v = [np.repeat(np.arange(n_v), 4)] + [rng.permutation(n_v)[:deg] for _ in range(hubs)]
    key = np.unique(np.concatenate(u).astype(np.int64) * n_v + np.concatenate(v))
    key = key[rng.permutation(len(key))]
    return ((key // n_v).astype(np.int32), (key % n_v).astype(np.int32),
            rng.choice([-1, 1], len(key)).astype(np.int8))


# windows of 16,384 keys: one, a full one and a short one, two full ones and a
# short one; and hubs just below 2^16 runs, which are packed
@pytest.mark.parametrize("n_u,deg,windows", [(9001, 67000, 1), (18001, 65536, 2), (36000, 69999, 2), (18001, 65535, 0)])
def test_unpacked_items_are_split(dbbc, n_u, deg, windows):
    n_v, hubs = 70000, 3
    u, v, s = _wide_hubs(n_u, n_v, hubs, deg, n_u)
    r = vp_counts(n_u, n_v, u, v, s, per_vertex=True, per_edge=True)
    held = []
    with dbbc.Graph(n_u, n_v, u, v, s) as h:
        for flags in (0, dbbc.DBBC_OPT_HOST_PLAN, 0):  # (the host planner cuts no items into parts)
            c, bu, bv, uu, uv = h.count_per_vertex(flags=flags)
            held.append(h.stats()["device_bytes"])
            assert (c.balanced, c.unbalanced, c.total) == (r.balanced, r.unbalanced, r.total)
            for t, want in ((bu, r.bal_u), (bv, r.bal_v), (uu, r.unb_u), (uv, r.unb_v)):
                assert np.array_equal(t.cpu().numpy(), want)
        for flags in (0, dbbc.DBBC_OPT_WIDE_EDGES):
            c, be, ue = h.count_per_edge(flags=flags)
            assert np.array_equal(be.cpu().numpy(), r.bal_e) and np.array_equal(ue.cpu().numpy(), r.unb_e)
    # the counters of the split hubs' windows, up to 128 KiB each (beside them
    # the two planners' lists differ by less than three windows)
    window = 4 * min(2 * n_u, 32768)
    counters = held[0] - held[1]
    assert hubs * max(windows, 1) * window <= counters < hubs * (max(windows, 1) + 1) * window, held
