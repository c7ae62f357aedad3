"""The device planner where its chunks can go wrong: entry counts around a
chunk of 1,024, rows that end at, cross and span chunks, blocks of rows with
none of their entries, small items of all sizes and single-item groups.  Per
counting kernel the wedges and runs equal the host planner's, and all counts
(integers) equal the oracle's."""

import numpy as np
import pytest

from oracle import vp_counts

pytestmark = pytest.mark.gpu

SMALL = dict(window_L=256, reverse_L=64, hub_T=0, part_work=4096)
HUBS = dict(window_L=512, reverse_L=64, hub_T=128, part_work=4096, small_work=100)


@pytest.fixture(scope="module")
def dbbc():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    import paper_2609_21848_amd as mod
    mod.load()
    return mod


def _check(dbbc, n_u, n_v, u, v, opts, seed=0):
    key = np.unique(u.astype(np.int64) * n_v + v)
    u, v = (key // n_v).astype(np.int32), (key % n_v).astype(np.int32)
    s = np.random.default_rng(seed).choice([-1, 1], len(u)).astype(np.int8)
    r = vp_counts(n_u, n_v, u, v, s, per_vertex=True)
    with dbbc.Graph(n_u, n_v, u, v, s) as h:
        per = []
        for flags in (0, dbbc.DBBC_OPT_HOST_PLAN):
            c = h.count(flags=flags | dbbc.DBBC_OPT_TIME_KERNELS, **opts)
            assert tuple(c) == (r.balanced, r.unbalanced, r.total, r.wedges)
            per.append({k["name"]: (k["wedges"], k["segments"]) for k in h.kernel_times()
                        if k["name"] in ("direct", "reverse", "small", "hash")})
        assert per[0] == per[1]
        c, bu, bv, uu, uv = h.count_per_vertex(**opts)
        for t, want in ((bu, r.bal_u), (bv, r.bal_v), (uu, r.unb_u), (uv, r.unb_v)):
            assert np.array_equal(t.cpu().numpy(), want)


@pytest.mark.parametrize("m", [1, 2, 255, 256, 1023, 1024, 1025, 2047, 2048, 2049, 5000])
@pytest.mark.parametrize("opts", [{}, SMALL])
def test_entries_around_chunks(dbbc, m, opts):
    n_u, n_v = 400, 300
    key = np.random.default_rng(m).choice(n_u * n_v, m, replace=False)
    _check(dbbc, n_u, n_v, key // n_v, key % n_v, opts)


@pytest.mark.parametrize("degrees", [[1024] * 6, [1023, 1, 1025, 1, 2048, 3], [5000, 3000, 1] + [2] * 900,
                                     [3000] * 40 + [600] * 500])
@pytest.mark.parametrize("opts", [{}, SMALL, HUBS])
def test_rows_that_end_at_and_span_chunks(dbbc, degrees, opts):
    rng = np.random.default_rng(len(degrees))
    n_v = 6000
    u = np.repeat(np.arange(len(degrees)), degrees)
    v = np.concatenate([np.sort(rng.choice(n_v, d, replace=False)) // (1 if d > 700 else 8) for d in degrees])
    _check(dbbc, len(degrees) + 5, n_v, u, v, opts)


@pytest.mark.parametrize("opts", [{}, SMALL, dict(SMALL, small_work=512), HUBS])
def test_small_items_of_all_sizes_and_sparse_sides(dbbc, opts):
    # mids of degree 2 .. 60 over rows of very different lengths, and most
    # vertices of both sides without an edge
    rng = np.random.default_rng(7)
    n_u, n_v = 9000, 7000
    u, v = [], []
    for y in range(1500):
        d = 2 + y % 59
        u.append(rng.choice(700 if y % 3 else 60, min(d, 60), replace=False))
        v.append(np.full(len(u[-1]), y * 4))
    _check(dbbc, n_u, n_v, np.concatenate(u), np.concatenate(v), opts)


@pytest.mark.parametrize("swap", [False, True])
@pytest.mark.parametrize("part_work", [4096, 20000])
def test_parts_of_rows_whose_mids_are_far_larger(dbbc, swap, part_work):
    # 900 rows of degree 12 to 20 through 40 mids of some hundred entries: heavy
    # items whose own side has small degrees only
    rng = np.random.default_rng(5)
    u = np.repeat(np.arange(900), 12 + np.arange(900) % 9)
    v = np.concatenate([rng.choice(40, 12 + x % 9, replace=False) for x in range(900)])
    n = (900, 40)
    if swap:
        u, v, n = v, u, n[::-1]
    _check(dbbc, *n, u, v, dict(part_work=part_work, small_work=2, hub_T=0, window_L=1024, reverse_L=64))
