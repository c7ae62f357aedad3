"""Per-vertex and per-edge passes on reverse items around the sizes at which a
walk takes another step: 64 runs a batch, 256 staged entries a round and the
rounds that stay in registers, long runs of whole and part chunks, and the run
count past which an endpoint is a direct item.  Every vertex's and edge's counts
(integers) must equal the oracle's."""

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


def _endpoints(keys, mids, degrees, seed):
    """`keys` top vertices over mids of growing row length (runs of 1 to `keys`
    entries), and endpoints of the given degrees."""
    rng = np.random.default_rng(seed)
    mu, kv = np.nonzero(rng.random((mids, keys)) < (np.arange(mids)[:, None] + 1) / mids)
    u, v = [mu], [kv]
    for i, d in enumerate(degrees):
        u.append(rng.choice(mids, d, replace=False))
        v.append(np.full(d, keys + i))
    u, v = np.concatenate(u), np.concatenate(v)
    order = rng.permutation(len(u))
    return (u[order].astype(np.int32), v[order].astype(np.int32),
            rng.choice([-1, 1], len(u)).astype(np.int8))


@pytest.mark.parametrize("keys,mids", [(256, 1024), (512, 1024), (1280, 1200), (4096, 1100)])
@pytest.mark.parametrize("long_len", [16, 128, 4096])
def test_reverse_items_of_every_step(dbbc, keys, mids, long_len):
    degrees = [d for d in (2, 8, 31, 63, 64, 65, 100, 127, 128, 129, 192, 193, 254, 255, 256) for _ in range(3)]
    u, v, s = _endpoints(keys, mids, degrees, keys + long_len)
    n_v = keys + len(degrees)
    r = vp_counts(mids, n_v, u, v, s, per_vertex=True, per_edge=True)
    opts = dict(window_L=keys, reverse_L=keys, hub_T=0, long_len=long_len)
    with dbbc.Graph(mids, n_v, u, v, s) as h:
        c, bu, bv, uu, uv = h.count_per_vertex(**opts)
        assert (c.balanced, c.unbalanced, c.total) == (r.balanced, r.unbalanced, r.total)
        for t, want in ((bu, r.bal_u), (bv, r.bal_v), (uu, r.unb_u), (uv, r.unb_v)):
            assert np.array_equal(t.cpu().numpy(), want)
        for flags in (0, dbbc.DBBC_OPT_WIDE_EDGES):
            c, be, ue = h.count_per_edge(flags=flags, **opts)
            assert np.array_equal(be.cpu().numpy(), r.bal_e) and np.array_equal(ue.cpu().numpy(), r.unb_e)


def test_light_reverse_items(dbbc):
    """Endpoints of 60 to 194 wedges in runs of 1 to 64 entries: on either side of
    the work up to which a reverse item is a small one."""
    rng = np.random.default_rng(5)
    keys, lengths, copies = 256, (1, 2, 4, 8, 16, 32, 64), 200
    u, v, n_u = [], [], 300
    u.append(np.repeat(np.arange(n_u), keys))  # every key is adjacent to these
    v.append(np.tile(np.arange(keys), n_u))
    n_v = keys
    for length in lengths:
        mids = n_u + np.arange(copies)
        n_u += copies
        u.append(np.repeat(mids, length))
        v.append(np.tile(np.arange(length), copies))
        for work in (60, 63, 64, 65, 66, 128, 190, 191, 192, 193, 194):
            d = work // length
            u.append(rng.choice(mids, d, replace=False))
            v.append(np.full(d, n_v))
            n_v += 1
    u, v = np.concatenate(u), np.concatenate(v)
    order = rng.permutation(len(u))
    u, v = u[order].astype(np.int32), v[order].astype(np.int32)
    s = rng.choice([-1, 1], len(u)).astype(np.int8)
    r = vp_counts(n_u, n_v, u, v, s, per_vertex=True, per_edge=True)
    with dbbc.Graph(n_u, n_v, u, v, s) as h:
        for small_work in (-1, 2, 64, 100):
            opts = dict(window_L=keys, reverse_L=keys, hub_T=0, small_work=small_work)
            c = h.count(**opts)
            assert (c.balanced, c.unbalanced, c.total) == (r.balanced, r.unbalanced, r.total)
            c, bu, bv, uu, uv = h.count_per_vertex(**opts)
            for t, want in ((bu, r.bal_u), (bv, r.bal_v), (uu, r.unb_u), (uv, r.unb_v)):
                assert np.array_equal(t.cpu().numpy(), want)
            c, be, ue = h.count_per_edge(**opts)
            assert np.array_equal(be.cpu().numpy(), r.bal_e) and np.array_equal(ue.cpu().numpy(), r.unb_e)
