"""The work that users of this library have it do, as measurable cases.

A case is a dict of plain values; its ``use`` says which calls make up one pass:

  pass      walks + RPE table of a seed list (fused call), then the union join of a query list
  ids       Algorithm 1 end to end (walks, table of RPE-IDs, pruned array), then the join over IDs
  calls     sample_walks and build_rpe as two calls, the sizes counted by the library
  online    a resident graph, a batch of new queries: walks + RPE of their nodes only, then the join
  lookup    a resident table, one training batch of queries joined
  ship      a resident table with RPE-IDs: the per-walk-position IDs of a query list
  prune     a resident table pruned to its distinct count vectors
  batches   a query list: its incidence lists, then mini-batches by breadth-first search

Graphs and queries have the shapes of ``paper_2202_13538_amd/synth.py`` (Chung-Lu and R-MAT
graphs with shuffled node ids, uniform tuples, half edges and half random pairs), drawn on the
GPU so that making them is quick.  All results are whole numbers and the random stream is
counter-based, so every output is compared exactly.

Outputs whose size depends on the data go to buffers of the worst case's size, allocated once, as
288 GB of device memory allow; what a pass leaves unwritten there is zero.
"""
from __future__ import annotations

import torch

from paper_2202_13538_amd import binding

_context = None


def _ctx() -> binding.Context:
    """The one context that a program keeps (its workspaces only grow)."""
    global _context
    if _context is None:
        _context = binding.Context()
    return _context


# --------------------------------------------------------------------------- #
# cases
# --------------------------------------------------------------------------- #
def listed() -> list[dict]:
    return [
        # the smallest whole pass: launches and read-backs count (a first try of the library, a
        # unit test, a toy graph)
        dict(name="smoke_pass", use="pass", graph="rmat", nodes=4096, edges=32_768, gamma=0.0,
             M=50, m=4, queries=1024, k=2),
        # a medium graph with many walks per node: every node's table, one epoch of link queries
        dict(name="collab_pass", use="pass", graph="chung_lu", nodes=235_000, edges=1_300_000,
             gamma=2.1, M=200, m=4, queries=65_536, k=2),
        # the benchmark's workload: preprocessing of a 2.9M-node graph and a million link queries
        dict(name="citation_pass", use="pass", graph="chung_lu", nodes=2_900_000,
             edges=30_000_000, gamma=2.3, M=100, m=4, queries=1_048_576, k=2),
        # higher-order prediction: triples
        dict(name="triples_pass", use="pass", graph="chung_lu", nodes=1_000_000,
             edges=10_000_000, gamma=2.2, M=100, m=3, queries=262_144, k=3),
        # longer walks than usual, an odd number of them on an odd number of nodes
        dict(name="long_walks_pass", use="pass", graph="chung_lu", nodes=99_991, edges=800_003,
             gamma=2.3, M=61, m=9, queries=30_011, k=2),
        # a dense graph, the table kept as RPE-IDs with the distinct vectors stored once
        dict(name="ppa_ids", use="ids", graph="rmat", nodes=1 << 19, edges=21_000_000, gamma=0.0,
             M=200, m=3, queries=262_144, k=2),
        # walks and table as two calls (a program that keeps the walks for other uses as well)
        dict(name="two_calls", use="calls", graph="chung_lu", nodes=500_009, edges=4_000_000,
             gamma=2.3, M=50, m=4),
        # serving: 1,000 link queries that arrive on a 2.9M-node graph
        dict(name="online_queries", use="online", graph="chung_lu", nodes=2_900_000,
             edges=30_000_000, gamma=2.3, M=100, m=4, queries=1000, k=2),
        # one training step of the paper's default batch size on a resident table
        dict(name="training_batch", use="lookup", graph="chung_lu", nodes=235_000,
             edges=1_300_000, gamma=2.1, M=200, m=4, queries=32, k=2),
        # the form of the join that is shipped to a neural encoder: RPE-IDs of walk positions
        dict(name="ship_ids", use="ship", graph="chung_lu", nodes=235_000, edges=1_300_000,
             gamma=2.1, M=200, m=4, queries=65_536, k=2),
        # a finished table pruned afterwards
        dict(name="prune_table", use="prune", graph="chung_lu", nodes=1_000_000,
             edges=10_000_000, gamma=2.2, M=50, m=4),
        # mini-batches for training with the default limits
        dict(name="mini_batches", use="batches", nodes=2_900_000, edges=30_000_000, gamma=2.3,
             queries=1_048_576, k=2, batches=8192, start=16, B1=1500, B2=32),
    ]


def _log_uniform(rng, low: int, high: int) -> int:
    return int(round(low * (high / low) ** rng.random()))


def draw(rng) -> dict:
    use = rng.choice(["pass", "pass", "pass", "ids", "calls", "online", "lookup", "ship", "prune",
                      "batches"])
    k = rng.choice([2, 2, 3])
    if use == "batches":
        B2 = _log_uniform(rng, 16, 4096)
        wanted = _log_uniform(rng, 131_072, 524_288)  # queries in all batches together
        return dict(use=use, nodes=_log_uniform(rng, 200_000, 2_900_000), edges=30_000_000,
                    gamma=round(rng.uniform(2.1, 2.5), 2),
                    queries=_log_uniform(rng, 65_536, 1_048_576), k=k,
                    batches=max(16, wanted // B2), start=16, B1=B2 * rng.choice([k, 47]), B2=B2)
    # the calls that prune are for walks whose count vectors repeat: up to four steps
    m = rng.choice([2, 3, 3, 4, 4, 4] + ([] if use in ("ids", "ship", "prune") else [5, 6, 9]))
    M = min(_log_uniform(rng, 20, 200), 2048 // (m + 1))
    rows, vector = 1 + M * m, 2 * (m + 1)  # of a table block, at most; bytes of a count vector
    bound = {"pass": 22e9, "ids": 12e9, "calls": 8e9, "online": 1e12, "lookup": 6e9, "ship": 6e9,
             "prune": 8e9}[use]
    low = 200_000 if use == "online" else 4096
    nodes = min(_log_uniform(rng, low, 2_900_000),
                int(bound / (4 * M * (m + 1) + rows * (4 + vector))))
    case = dict(use=use, graph="chung_lu", nodes=nodes, gamma=round(rng.uniform(2.1, 2.5), 2))
    if rng.random() < 0.3:
        case.update(graph="rmat", nodes=1 << (nodes.bit_length() - 1), gamma=0.0)
    case.update(edges=min(int(case["nodes"] * rng.uniform(4, 40)), 30_000_000), M=M, m=m)
    row = k * rows * (4 + k * vector)  # bytes of a query's joined rows, at most
    if use == "pass":
        case.update(queries=min(_log_uniform(rng, 1000, 1_048_576), int(18e9 / row)), k=k)
    elif use == "ids":
        case.update(queries=min(_log_uniform(rng, 1000, 500_000), int(10e9 / row)), k=k)
    elif use == "online":
        case.update(queries=_log_uniform(rng, 32, 5000), k=k)
    elif use == "lookup":
        case.update(queries=_log_uniform(rng, 16, 8192), k=k)
    elif use == "ship":
        case.update(queries=min(_log_uniform(rng, 1000, 262_144), int(8e9 / row)), k=k)
    return case


# --------------------------------------------------------------------------- #
# inputs
# --------------------------------------------------------------------------- #
class _Endpoints:
    """Endpoints with Chung-Lu weights (i + i0)^(-1/(gamma-1)), by the inverse of the weights'
    integral; i0 makes the largest expected degree about sqrt(2 * edges)."""

    def __init__(self, n: int, edges: int, gamma: float):
        self.n, self.p = n, 1.0 - 1.0 / (gamma - 1.0)

        def top_degree(i0: float) -> float:
            total = ((n + i0) ** self.p - i0 ** self.p) / self.p
            return 2.0 * edges * i0 ** (self.p - 1.0) / total

        low, high = 1e-3, float(n)
        for _ in range(60):
            mid = 0.5 * (low + high)
            low, high = (mid, high) if top_degree(mid) > (2.0 * edges) ** 0.5 else (low, mid)
        self.i0 = high

    def __call__(self, count: int, g) -> torch.Tensor:
        u = torch.rand(count, dtype=torch.float64, device="cuda", generator=g)
        a, b = self.i0 ** self.p, (self.n + self.i0) ** self.p
        return ((a + u * (b - a)) ** (1.0 / self.p) - self.i0).long().clamp_(0, self.n - 1)


def _rmat_pairs(scale: int, count: int, g):
    """R-MAT with quadrant probabilities 0.57, 0.19, 0.19, 0.05."""
    u = torch.zeros(count, dtype=torch.int64, device="cuda")
    v = torch.zeros_like(u)
    for _ in range(scale):
        r = torch.rand(count, device="cuda", generator=g)
        u = u * 2 + (r >= 0.76)
        v = v * 2 + (((r >= 0.57) & (r < 0.76)) | (r >= 0.95))
    return u, v


def _graph(case: dict, g):
    """(row_ptr, col_idx) int32: `edges` distinct undirected edges, both directions of each, rows
    ascending, node ids shuffled."""
    n, want = case["nodes"], min(case["edges"], case["nodes"] * (case["nodes"] - 1) // 8)
    ends = _Endpoints(n, want, case["gamma"]) if case["graph"] == "chung_lu" else None
    keys = torch.empty(0, dtype=torch.int64, device="cuda")
    while keys.numel() < want:
        count = int((want - keys.numel()) * 1.2) + 1024
        u, v = (ends(count, g), ends(count, g)) if ends else _rmat_pairs(n.bit_length() - 1, count, g)
        new = (torch.minimum(u, v) * n + torch.maximum(u, v))[u != v]
        keys = torch.unique(torch.cat([keys, new]))
    keep = torch.randperm(keys.numel(), device="cuda", generator=g)[:want]
    keys = keys[keep]
    name = torch.randperm(n, device="cuda", generator=g)
    u, v = name[keys // n], name[keys % n]
    both = torch.sort(torch.cat([u * n + v, v * n + u])).values
    row_ptr = torch.searchsorted(both, torch.arange(n + 1, device="cuda") * n).int()
    return row_ptr, (both % n).int()


def _queries(case: dict, row_ptr, col_idx, g) -> torch.Tensor:
    """int32[queries][k]: pairs on Chung-Lu graphs are half edges and half random pairs, other
    tuples are uniform; the nodes of a tuple are distinct."""
    n, q, k = case["nodes"], case["queries"], case["k"]
    first = torch.randint(0, n, (q, 1), device="cuda", generator=g)
    step = torch.randint(1, (n - 1) // (k - 1) + 1, (q, k - 1), device="cuda", generator=g)
    tuples = torch.cat([first, (first + step.cumsum(1)) % n], dim=1)
    if k == 2 and case["graph"] == "chung_lu":
        e = torch.randint(0, col_idx.numel(), (q // 2,), device="cuda", generator=g)
        src = torch.searchsorted(row_ptr.long(), e, right=True) - 1
        tuples[: q // 2] = torch.stack([src, col_idx[e].long()], dim=1)
        tuples = tuples[torch.randperm(q, device="cuda", generator=g)]
    return tuples.int().contiguous()


class _State:
    pass


def prepare(case: dict, seed: int) -> _State:
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    s = _State()
    s.case, s.ctx, s.rng_seed = case, _ctx(), seed * 0x9E3779B97F4A7C15 % (1 << 64)
    if case["use"] == "batches":
        _prepare_batches(s, g)
        return s
    n, M, m = case["nodes"], case["M"], case["m"]
    s.row_ptr, s.col_idx = _graph(case, g)
    s.seeds = torch.arange(n, dtype=torch.int32, device="cuda")
    s.max_set = 1 + M * m
    if "queries" in case:
        s.queries = _queries(case, s.row_ptr, s.col_idx, g)
    if case["use"] == "online":
        # the nodes that the batch names, tuple after tuple: block 0, 1, .. of the table
        s.seeds = s.queries.flatten()
        s.queries = torch.arange(s.seeds.numel(), dtype=torch.int32, device="cuda").view(-1, case["k"])
    if case["use"] in ("lookup", "ship", "prune"):
        s.walks, s.rpe_off, s.rpe_ids, s.rpe_cnt = binding.sample_walks_rpe(
            s.ctx, s.row_ptr, s.col_idx, s.seeds, M, m, s.rng_seed)
    if case["use"] == "ship":
        _, s.code = binding.prune_rpe(s.ctx, s.rpe_cnt)
    _prepare_outputs(s)
    return s


def _zeros(dtype, *shape) -> torch.Tensor:
    return torch.zeros(shape, dtype=dtype, device="cuda")


def _prepare_outputs(s: _State) -> None:
    case, use = s.case, s.case["use"]
    n, M, L = s.seeds.numel(), case["M"], case["m"] + 1
    i32, i64, u16 = torch.int32, torch.int64, torch.uint16
    s.cap = binding.rpe_rows_bound(n, M, L - 1)
    if use in ("pass", "ids", "calls", "online"):
        s.walks = _zeros(i32, n, M, L)
        s.rpe_off, s.rpe_ids = _zeros(i64, n + 1), _zeros(i32, s.cap)
        s.rpe_cnt = None if use == "ids" else _zeros(u16, s.cap, L)
    if use == "calls":
        s.sizes = _zeros(i32, n)
    if use in ("ids", "prune"):
        s.cap_T = 1 << 20
        s.T, s.code = _zeros(u16, s.cap_T, L), _zeros(i32, s.cap)
    if use in ("pass", "ids", "online", "lookup"):
        q, k = s.queries.shape
        s.join_cap = q * k * s.max_set
        s.join_off, s.join_ids = _zeros(i64, q + 1), _zeros(i32, s.join_cap)
        s.join_cnt = _zeros(i32, s.join_cap, k) if use == "ids" else _zeros(u16, s.join_cap, k, L)
    if use == "ship":
        s.out = _zeros(i32, case["queries"], case["k"], M, L, case["k"])


def _prepare_batches(s: _State, g) -> None:
    case = s.case
    n, q, k, b = case["nodes"], case["queries"], case["k"], case["batches"]
    # half of the tuples are made of well-connected nodes, as the ends of edges are
    ends = _Endpoints(n, case["edges"], case["gamma"])
    name = torch.randperm(n, device="cuda", generator=g)
    tuples = torch.randint(0, n, (q, k), device="cuda", generator=g)
    tuples[: q // 2] = name[ends((q // 2) * k, g)].view(-1, k)
    s.queries = tuples[torch.randperm(q, device="cuda", generator=g)].int().contiguous()
    # seed-sets are drawn from the nodes that queries name
    at = torch.randint(0, q * k, (b, case["start"]), device="cuda", generator=g)
    s.start = s.queries.view(-1)[at].contiguous()
    s.vbar, s.batch, s.tuples, s.counts = (
        torch.full(shape, -1, dtype=torch.int32, device="cuda")
        for shape in ((b, case["B1"]), (b, case["B2"]), (b, case["B2"], k), (b, 2)))


# --------------------------------------------------------------------------- #
# one pass
# --------------------------------------------------------------------------- #
def _counts(t: torch.Tensor) -> torch.Tensor:
    return t.view(torch.int16)  # the same bits in a type that every torch operation knows


def _ok(rc: int) -> None:
    if rc != binding.OK:
        raise binding.SurelError(rc, "perf case")


def _join(s: _State):
    rc, rows = binding.join_queries_raw(s.ctx, s.rpe_off, s.rpe_ids, s.rpe_cnt, s.queries, s.max_set,
                                        s.join_cap, s.join_off, s.join_ids, s.join_cnt)
    _ok(rc)
    return rows, s.join_off, s.join_ids, _counts(s.join_cnt)


def run(s: _State):
    case, ctx = s.case, s.ctx
    use = case["use"]
    if use == "batches":
        inc_off, inc_q = binding.query_incidence(ctx, s.queries, case["nodes"])
        _ok(binding.bfs_batches_raw(ctx, s.queries, case["nodes"], inc_off, inc_q, s.start,
                                    case["B1"], case["B2"], s.vbar, s.batch, s.tuples, s.counts))
        return inc_off, inc_q, s.vbar, s.batch, s.tuples, s.counts
    M, m = case["M"], case["m"]
    if use in ("pass", "online"):
        rc, rows = binding.sample_walks_rpe_raw(ctx, s.row_ptr, s.col_idx, s.seeds, M, m, s.rng_seed,
                                                s.walks, s.cap, s.rpe_off, s.rpe_ids, s.rpe_cnt)
        _ok(rc)
        return (s.walks, rows, s.rpe_off, s.rpe_ids, _counts(s.rpe_cnt)) + _join(s)
    if use == "ids":
        rc, rows, n_T = binding.sample_walks_rpe_ids_raw(
            ctx, s.row_ptr, s.col_idx, s.seeds, M, m, s.rng_seed, s.walks, s.cap, s.rpe_off,
            s.rpe_ids, None, s.code, s.cap_T, s.T)
        _ok(rc)
        rc, joined = binding.join_query_ids_raw(ctx, s.rpe_off, s.rpe_ids, s.code, s.queries,
                                                s.max_set, s.join_cap, s.join_off, s.join_ids,
                                                s.join_cnt)
        _ok(rc)
        return (s.walks, rows, s.rpe_off, s.rpe_ids, s.code, n_T, _counts(s.T), joined, s.join_off,
                s.join_ids, s.join_cnt)
    if use == "calls":
        binding.sample_walks(ctx, s.row_ptr, s.col_idx, s.seeds, M, m, s.rng_seed, out=s.walks,
                             set_sizes=s.sizes)
        rc, rows = binding.build_rpe_raw(ctx, s.walks, case["nodes"], s.cap, s.rpe_off, s.rpe_ids,
                                         s.rpe_cnt, set_sizes=s.sizes)
        _ok(rc)
        return s.walks, s.sizes, rows, s.rpe_off, s.rpe_ids, _counts(s.rpe_cnt)
    if use == "lookup":
        return _join(s)
    if use == "ship":
        return binding.query_rpe_ids(ctx, s.walks, s.rpe_off, s.rpe_ids, s.queries, s.max_set,
                                     out=s.out, code=s.code)
    if use == "prune":
        rc, n_T = binding.prune_rpe_raw(ctx, s.rpe_cnt, s.cap_T, s.T, s.code)
        _ok(rc)
        return n_T, _counts(s.T), s.code
    raise ValueError(use)


# --------------------------------------------------------------------------- #
# what a pass cannot do without
# --------------------------------------------------------------------------- #
#: Distinct nodes of a seed's walks over the M*m steps, and rows of a union over those of its
#: blocks, as they come out on these graphs (the exact numbers depend on the draw).
DISTINCT, UNION = 0.7, 0.97


def work(case: dict) -> dict:
    """Inputs read once (of the graph no more than 12 bytes a step), outputs written once; the
    operations are the ten rounds of the generator per four steps, and one per value moved."""
    use = case["use"]
    q, k = case.get("queries", 0), case.get("k", 2)
    if use == "batches":
        b = case["batches"]
        entries = q * k
        out = b * (min(case["B1"], case["B2"] * k + case["start"]) + case["B2"] * (1 + k) + 2)
        moved = entries * 4 * 2 + (case["nodes"] + 1) * 8 + b * case["start"] * 4 + out * 4
        return {"bytes": moved, "flops": moved / 4}
    M, m = case["M"], case["m"]
    L = m + 1
    seeds = min(q * k, case["nodes"]) if use == "online" else case["nodes"]
    block = 1 + DISTINCT * M * m                        # table rows of a seed
    vector = 4 if use == "ids" else 2 * L
    total = 0.0
    if use in ("pass", "ids", "calls", "online"):       # walks and table
        graph = 4 * (case["nodes"] + 1) + 8 * case["edges"]
        total += min(graph, 12 * seeds * M * m) + 4 * seeds + 4 * seeds * M * L
        total += 8 * seeds + seeds * block * (4 + vector)
        total += 4 * seeds if use == "calls" else 0
    if use in ("pass", "ids", "online", "lookup"):      # join: the blocks that are named, once
        total += min(q * k, seeds) * (16 + block * (4 + vector)) + q * k * 4
        total += q * 8 + q * k * block * UNION * (4 + k * vector)
    if use == "ship":
        total += min(q * k, seeds) * (16 + block * 8 + 4 * M * L) + q * k * 4
        total += 4 * q * k * M * L * k
    if use == "prune":
        total += seeds * block * (2 * L + 4)
    steps = seeds * M * m if use in ("pass", "ids", "calls", "online") else 0
    return {"bytes": total, "flops": total / 4 + 20 * steps}


def tolerance(case: dict):
    return "exact"
