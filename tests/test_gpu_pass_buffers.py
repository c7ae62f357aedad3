"""What the per-vertex and the per-edge pass keep on a handle: each its own
credits (the per-edge pass none per vertex), whichever comes first, and both
give the oracle's counts in either order."""

import numpy as np
import pytest

from oracle import vp_counts
from synth import chung_lu_graph

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("opts", [{}, dict(hub_T=256)])
@pytest.mark.parametrize("order", ["ev", "ve", "evev", "veve"])
def test_passes_keep_their_own_buffers(order, opts):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    import paper_2609_21848_amd as dbbc
    g = chung_lu_graph(3000, 2000, 40000, 2.1, 1.9, 0.4, seed=11)
    r = vp_counts(g.n_u, g.n_v, g.u, g.v, g.sign, per_vertex=True, per_edge=True)
    per_vertex = 32 * (g.n_u + g.n_v) + (1 << 20)  # four words a vertex, and the key sums
    per_edge = 48 * g.m + 4 * g.m                  # six words an edge, and a map
    with dbbc.Graph(g.n_u, g.n_v, g.u, g.v, g.sign) as h:
        held, seen = h.stats()["device_bytes"], set()
        for k, p in enumerate(order):
            if p == "v":
                c, bu, bv, uu, uv = h.count_per_vertex(**opts)
                for t, want in ((bu, r.bal_u), (bv, r.bal_v), (uu, r.unb_u), (uv, r.unb_v)):
                    assert np.array_equal(t.cpu().numpy(), want)
            else:
                c, be, ue = h.count_per_edge(**opts)
                assert np.array_equal(be.cpu().numpy(), r.bal_e) and np.array_equal(ue.cpu().numpy(), r.unb_e)
            assert (c.balanced, c.unbalanced, c.total) == (r.balanced, r.unbalanced, r.total)
            now = h.stats()["device_bytes"]
            if k > 0:  # (the first pass makes the plan too)
                assert now - held == (0 if p in seen else per_vertex if p == "v" else per_edge)
            held = now
            seen.add(p)
