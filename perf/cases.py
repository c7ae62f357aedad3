"""What a user of this framework has it do, as timed cases.

A case is one operation on one graph (or one batch of small graphs):

* ``count``: the exact count of a resident, planned graph (a serving loop or
  a bench step: the handle and its plan are kept, the count is repeated);
* ``vertices`` / ``edges``: the per-vertex and per-edge counts of a resident
  graph (features for every vertex or interaction of the graph);
* ``create``: a new graph from its edge list to its first count (build, plan,
  count), from device tensors or from host arrays, as an upload is answered;
* ``text``: the same from an edge-list text, raw ids and all;
* ``batch``: many small resident graphs counted by one captured launch
  sequence.

Graphs are drawn on the GPU from the seed alone: Chung-Lu pairs (per side,
Pareto weights of exponent ``gamma_*`` clipped so that no expected degree
passes the cap, the first ``m`` distinct pairs in draw order), or uniform
pairs where ``gamma`` is 0; a sign is -1 with probability ``q``.  ``repeat``
gives the share of further records that repeat an earlier pair with a new
sign (the last record wins).
"""

from __future__ import annotations

import math

import numpy as np
import torch

import paper_2609_21848_amd as dbbc

# the largest number of wedges whose counts are also formed in plain torch
EXACT_WEDGES = 250_000_000


def _case(op, n_u, n_v, m, gamma_u, gamma_v, q, cap=0, repeat=0.0, where="device", graphs=1, name=None):
    c = dict(op=op, n_u=n_u, n_v=n_v, m=m, gamma_u=gamma_u, gamma_v=gamma_v, q=q, cap=cap, repeat=repeat,
             where=where, graphs=graphs)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest calls: a repeated count of a 20,000-edge graph (the
        # paper's smallest datasets), and such a graph's upload to its count
        _case("count", 2_000, 1_500, 20_000, 0.0, 0.0, 0.3, name="count_20k"),
        _case("create", 2_000, 1_500, 20_000, 0.0, 0.0, 0.3, name="create_20k"),
        # ordinary ones: 2M edges (the paper's middle datasets), resident,
        # uploaded from host arrays with repeated records, and read from text
        _case("count", 200_000, 100_000, 2_000_000, 2.3, 2.1, 0.25, name="count_2m"),
        _case("create", 200_000, 100_000, 2_000_000, 2.3, 2.1, 0.25, repeat=0.1, where="host",
              name="create_2m_host"),
        _case("text", 200_000, 100_000, 2_000_000, 2.3, 2.1, 0.25, name="text_2m"),
        # the benchmark's workload: 50M edges, repeated counts and an upload
        _case("count", 5_000_000, 2_000_000, 50_000_000, 2.1, 1.9, 0.4, cap=100_000, name="count_50m"),
        _case("create", 5_000_000, 2_000_000, 50_000_000, 2.1, 1.9, 0.4, cap=100_000, name="create_50m"),
        # per-vertex counts of a ragged middle-sized graph and of the
        # benchmark's; per-edge counts of the middle dataset and a larger one
        _case("vertices", 33_331, 16_661, 333_667, 2.2, 2.2, 0.3, name="vertices_333k"),
        _case("vertices", 5_000_000, 2_000_000, 50_000_000, 2.1, 1.9, 0.4, cap=100_000, name="vertices_50m"),
        _case("edges", 200_000, 100_000, 2_000_000, 2.3, 2.1, 0.25, name="edges_2m"),
        _case("edges", 2_000_000, 1_000_000, 20_000_000, 2.2, 2.0, 0.3, cap=100_000, name="edges_20m"),
        # a server's full batch of small graphs (200 to 50,000 edges each)
        _case("batch", 5_000, 5_000, 50_000, 2.2, 2.2, 0.3, graphs=512, name="batch_512"),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    op = rng.choice(["count", "create", "create", "text", "vertices", "edges", "batch"])
    if op == "batch":
        return _case(op, log_int(500, 5_000), log_int(500, 5_000), log_int(2_000, 50_000),
                     rng.choice([0.0, 2.2, 2.5]), 2.2, rng.uniform(0.1, 0.5), graphs=log_int(16, 512))
    m = log_int(1_000, {"count": 40e6, "create": 40e6, "text": 8e6, "vertices": 30e6, "edges": 15e6}[op])
    n_u = max(40, int(m * rng.uniform(0.05, 0.2)))
    n_v = max(30, int(n_u * rng.uniform(0.3, 1.1)))
    m = min(m, n_u * n_v // 3)
    # heavy tails as in the listed cases; the largest graphs stay below the
    # benchmark workload's skew
    lo = 2.0 if m < 5_000_000 else 2.1
    uniform = rng.random() < 0.15
    gu = 0.0 if uniform else rng.uniform(lo + 0.05, 2.8)
    gv = 0.0 if uniform else rng.uniform(lo, 2.6)
    where = rng.choice(["device", "host"]) if op == "create" and m < 10_000_000 else "device"
    repeat = rng.choice([0.0, 0.1, 0.5]) if op in ("create", "text", "edges") and m < 10_000_000 else 0.0
    return _case(op, n_u, n_v, m, gu, gv, rng.uniform(0.1, 0.9), cap=100_000, repeat=repeat, where=where)


# ---- inputs ------------------------------------------------------------------

def _picker(n, gamma, m, cap, gen):
    """A function of k: k vertex ids drawn by their Chung-Lu weights."""
    dev = gen.device
    if gamma == 0.0:
        return lambda k: torch.randint(n, (k,), generator=gen, device=dev)
    w = (1.0 - torch.rand(n, generator=gen, device=dev, dtype=torch.float64)).pow(-1.0 / (gamma - 1.0))
    w = torch.minimum(w, w.sum() * (cap / m))
    cdf = torch.cumsum(w, 0)
    cdf /= cdf[-1].clone()
    return lambda k: torch.searchsorted(
        cdf, torch.rand(k, generator=gen, device=dev, dtype=torch.float64)).clamp_(max=n - 1)


def _edges(c, gen):
    """(u, v, sign) of one graph: int32, int32 and int8 CUDA tensors."""
    n_u, n_v, m = c["n_u"], c["n_v"], c["m"]
    pick_u = _picker(n_u, c["gamma_u"], m, min(n_v, c["cap"] or n_v), gen)
    pick_v = _picker(n_v, c["gamma_v"], m, min(n_u, c["cap"] or n_u), gen)
    keys = torch.empty(0, dtype=torch.int64, device=gen.device)
    first = keys
    k = int(m * 1.2) + 64
    while True:
        keys = torch.cat([keys, pick_u(k) * n_v + pick_v(k)])
        ordered, at = torch.sort(keys, stable=True)
        head = torch.ones_like(ordered, dtype=torch.bool)
        head[1:] = ordered[1:] != ordered[:-1]
        first = at[head]
        if first.numel() >= m:
            break
        k = max(2 * (m - first.numel()), keys.numel() // 2)
    key = keys[torch.sort(first).values[:m]]
    if c["repeat"] > 0:
        more = key[torch.randint(m, (int(m * c["repeat"]),), generator=gen, device=gen.device)]
        key = torch.cat([key, more])
    sign = 1 - 2 * (torch.rand(key.numel(), generator=gen, device=gen.device) < c["q"]).to(torch.int8)
    return (key // n_v).to(torch.int32), (key % n_v).to(torch.int32), sign


def _text_edges(c, gen):
    """The records of a text: _edges', after one record for every vertex (a
    text names only vertices that have one)."""
    k = torch.arange(max(c["n_u"], c["n_v"]), device=gen.device, dtype=torch.int32)
    u, v, s = _edges(c, gen)
    return (torch.cat([k % c["n_u"], u]), torch.cat([k % c["n_v"], v]),
            torch.cat([torch.ones_like(k, dtype=torch.int8), s]))


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _batch_edges(c, gen):
    """The batch's graphs: sizes spread below the case's, as (n_u, n_v, u, v, sign)."""
    out = []
    share = torch.rand((c["graphs"], 3), generator=gen, device=gen.device).tolist()
    for a, b, e in share:
        n_u, n_v = max(50, int(c["n_u"] * a)), max(50, int(c["n_v"] * b))
        m = min(max(200, int(c["m"] * e)), n_u * n_v // 3)
        out.append((n_u, n_v, *_edges(dict(c, n_u=n_u, n_v=n_v, m=m), gen)))
    return out


# raw ids of a text's vertices: an odd multiplier below 2^34, so that ids of
# one to eleven digits occur in no order
_RAW_BITS = 34
_RAW_MUL = (2_654_435_761, 3_266_489_917)


def _raw(ids, side):
    return ((ids.to(torch.int64) + 1) * _RAW_MUL[side]) % (1 << _RAW_BITS)


def _text(u, v, sign):
    """The records as lines "u v s" (s = 1 positive, 0 negative), ids without
    leading zeros, as a uint8 CUDA tensor."""
    m, dev = u.numel(), u.device
    width = 11
    line = torch.empty((m, 2 * width + 4), dtype=torch.uint8, device=dev)
    keep = torch.ones_like(line, dtype=torch.bool)
    for side, ids in enumerate((u, v)):
        x = _raw(ids, side)
        at = side * (width + 1)
        for d in range(width):
            p = 10 ** (width - 1 - d)
            line[:, at + d] = (x // p % 10 + 48).to(torch.uint8)
            if p > 1:
                keep[:, at + d] = x >= p
        line[:, at + width] = 32
    line[:, 2 * width + 2] = torch.where(sign > 0, 49, 48).to(torch.uint8)
    line[:, 2 * width + 3] = 10
    return line[keep]


def prepare(case, seed):
    gen = _generator(seed)
    op = case["op"]
    if op == "batch":
        graphs = [dbbc.Graph(n_u, n_v, u, v, s) for n_u, n_v, u, v, s in _batch_edges(case, gen)]
        return dict(op=op, batch=dbbc.Batch(graphs, capture=True))
    u, v, s = _text_edges(case, gen) if op == "text" else _edges(case, gen)
    if op == "text":
        return dict(op=op, text=_text(u, v, s))
    if op == "create":
        if case["where"] == "host":
            u, v, s = (t.cpu().numpy() for t in (u, v, s))
        return dict(op=op, args=(case["n_u"], case["n_v"], u, v, s))
    g = dbbc.Graph(case["n_u"], case["n_v"], u, v, s)
    if op == "count":
        dbbc.dbbc_graph_plan(g.handle)
    return dict(op=op, graph=g)


def _stats(g):
    s = g.stats()
    return tuple(s[k] for k in ("n_u", "n_v", "m", "dups_dropped", "max_deg_u", "max_deg_v", "pivots_active"))


def run(state):
    op = state["op"]
    if op == "count":
        return tuple(state["graph"].count())
    if op == "batch":
        return torch.tensor(state["batch"].count())
    if op == "vertices":
        c, *arrays = state["graph"].count_per_vertex()
        return (tuple(c), *arrays)
    if op == "edges":
        c, *arrays = state["graph"].count_per_edge()
        return (tuple(c), *arrays)
    if op == "create":
        with dbbc.Graph(*state["args"]) as g:
            return tuple(g.count()) + _stats(g)
    with dbbc.Graph.from_text(state["text"]) as g:
        return (tuple(g.count()) + _stats(g), g.raw_ids(0), g.raw_ids(1))


def work(case):
    """Bytes: the records (or the resident edges, id and sign in one word)
    read once, the results written once.  A count's other bound, one counter
    update per wedge, depends on the graph's degrees and is not in a case."""
    m, n = case["m"], case["n_u"] + case["n_v"]
    m_in = m + int(m * case["repeat"])
    op = case["op"]
    read = {"count": 4 * m, "vertices": 4 * m, "edges": 4 * m, "create": 9 * m_in,
            "text": 24 * (m_in + max(case["n_u"], case["n_v"])), "batch": 4 * m * case["graphs"] // 2}[op]
    write = {"vertices": 16 * n, "edges": 16 * m_in, "text": 8 * n}.get(op, 32 * case["graphs"])
    return {"bytes": read + write, "flops": 0}


# ---- the same results in plain torch -------------------------------------------

def _exact_graph(n_u, n_v, u, v, sign, want):
    """Counts of one edge list (duplicates: the last record wins), by the
    wedges of every pivot in plain int64 torch.  Returns a dict of totals and
    of the arrays that ``want`` names, or None when there are too many wedges."""
    u, v, sign = u.to(torch.int64), v.to(torch.int64), sign.to(torch.int64)
    dev, m_in = u.device, u.numel()
    order = torch.sort(u * n_v + v, stable=True)
    last = torch.ones(m_in, dtype=torch.bool, device=dev)
    last[:-1] = order.values[1:] != order.values[:-1]
    rec = order.indices[last]
    eu, ev, es = u[rec], v[rec] + n_u, sign[rec]
    m, n = rec.numel(), n_u + n_v
    deg = torch.bincount(torch.cat([eu, ev]), minlength=n)
    # the priority order: degree, then id, highest first
    by = torch.sort(deg * n + torch.arange(n, device=dev), descending=True).indices
    rank = torch.empty_like(by)
    rank[by] = torch.arange(n, device=dev)
    # rows of both sides by rank, neighbours in priority order
    a, b = torch.cat([rank[eu], rank[ev]]), torch.cat([rank[ev], rank[eu]])
    rows = torch.sort(a * n + b)
    a, b = rows.values // n, rows.values % n
    edge = rows.indices % m
    s = es[edge]
    start = torch.zeros(n + 1, dtype=torch.int64, device=dev)
    start[1:] = torch.cumsum(torch.bincount(a, minlength=n), 0)
    place = torch.empty(2 * m, dtype=torch.int64, device=dev)  # record's entry in U's row, then in V's
    place[rows.indices] = torch.arange(2 * m, device=dev)
    mate = torch.cat([place[m:], place[:m]])[rows.indices]  # the same edge in the other row
    down = torch.nonzero(b > a).flatten()  # pivot a, mid b
    length = start[b[down] + 1] - mate[down] - 1  # the entries of row b past a
    wedges = int(length.sum())
    if wedges > EXACT_WEDGES:
        return None
    first = torch.repeat_interleave(down, length)
    off = torch.cumsum(length, 0) - length
    second = torch.arange(wedges, device=dev) - torch.repeat_interleave(off - mate[down] - 1, length)
    sym = s[first] * s[second] > 0
    pair = torch.sort(a[first] * n + b[second])
    head = torch.ones(wedges, dtype=torch.bool, device=dev)
    if wedges:
        head[1:] = pair.values[1:] != pair.values[:-1]
    pid = torch.empty(wedges, dtype=torch.int64, device=dev)
    pid[pair.indices] = torch.cumsum(head, 0) - 1
    n_pairs = int(head.sum())
    p = torch.zeros(n_pairs, dtype=torch.int64, device=dev).index_add_(0, pid, sym.to(torch.int64))
    q = torch.zeros(n_pairs, dtype=torch.int64, device=dev).index_add_(0, pid, (~sym).to(torch.int64))
    bal, unb = p * (p - 1) // 2 + q * (q - 1) // 2, p * q
    x, w = pair.values[head] // n, pair.values[head] % n
    out = dict(m=m, wedges=wedges, deg=deg, active=int((torch.bincount(a[first], minlength=n) > 0).sum()),
               pair_vertex=by[x], bal=bal, unb=unb, pivot=by[a[down]], length=length)
    shares = [torch.where(sym, p[pid] - 1, q[pid] - 1), torch.where(sym, q[pid], p[pid])]
    if "vertices" in want:
        out["vertices"] = []
        for pairs, mids in ((bal, shares[0]), (unb, shares[1])):
            t = torch.zeros(n, dtype=torch.int64, device=dev)
            t.index_add_(0, x, pairs).index_add_(0, w, pairs).index_add_(0, b[first], mids)
            out["vertices"].append(t[rank])
    if "edges" in want:
        out["edges"] = []
        for share in shares:
            t = torch.zeros(m, dtype=torch.int64, device=dev)
            t.index_add_(0, edge[first], share).index_add_(0, edge[second], share)
            out["edges"].append(torch.zeros(m_in, dtype=torch.int64, device=dev).index_copy_(0, rec, t))
    return out


def _totals(r):
    b, un = int(r["bal"].sum()), int(r["unb"].sum())
    return (b, un, b + un, r["wedges"])


def exact(case, seed):
    gen = _generator(seed)
    op = case["op"]
    if op == "batch":
        # all graphs side by side in one: the priority order inside a graph
        # stays what it is alone (U ids before V ids)
        graphs = _batch_edges(case, gen)
        off_u = np.cumsum([0] + [g[0] for g in graphs])
        off_v = np.cumsum([0] + [g[1] for g in graphs])
        r = _exact_graph(int(off_u[-1]), int(off_v[-1]),
                         torch.cat([g[2].to(torch.int64) + int(o) for g, o in zip(graphs, off_u)]),
                         torch.cat([g[3].to(torch.int64) + int(o) for g, o in zip(graphs, off_v)]),
                         torch.cat([g[4] for g in graphs]), ())
        if r is None:
            return None
        dev = r["bal"].device
        owner = torch.cat([torch.repeat_interleave(torch.arange(len(graphs), device=dev),
                                                   torch.tensor(np.diff(o), device=dev)) for o in (off_u, off_v)])
        out = torch.zeros((len(graphs), 4), dtype=torch.int64, device=dev)
        out[:, 0].index_add_(0, owner[r["pair_vertex"]], r["bal"])
        out[:, 1].index_add_(0, owner[r["pair_vertex"]], r["unb"])
        out[:, 2] = out[:, 0] + out[:, 1]
        out[:, 3].index_add_(0, owner[r["pivot"]], r["length"])
        return out.cpu()
    u, v, s = _text_edges(case, gen) if op == "text" else _edges(case, gen)
    n_u, n_v, raws = case["n_u"], case["n_v"], ()
    if op == "text":  # ids by the order of the raw ids that occur
        raws, ids = zip(*(torch.unique(_raw(t, side), return_inverse=True) for side, t in enumerate((u, v))))
        u, v = ids
        n_u, n_v = (r.numel() for r in raws)
    r = _exact_graph(n_u, n_v, u, v, s, (op,))
    if r is None:
        return None
    if op == "count":
        return _totals(r)
    if op in ("vertices", "edges"):
        arrays = r[op]
        if op == "vertices":
            arrays = [t for a in arrays for t in (a[:n_u], a[n_u:])]
        return (_totals(r), *arrays)
    head = _totals(r) + (n_u, n_v, r["m"], u.numel() - r["m"], int(r["deg"][:n_u].max()), int(r["deg"][n_u:].max()),
                         r["active"])
    return head if op == "create" else (head, *raws)
