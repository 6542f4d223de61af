"""Parity of the HIP path with the CPU oracle, through the C ABI, on a real MI355X.

Bit-exact comparison of walks, RPE tables and joins, element by element, on small and
medium inputs (several tiles, ragged tails, the degenerate cases) and of the device-detected
problems.  The workloads at their full sizes are in test_gpu_full_size.py.
"""
import itertools
import os
import re

import numpy as np
import pytest
import torch

import oracle
from paper_2202_13538_amd import binding, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    assert torch.cuda.is_available(), "these tests need the GPU"
    assert os.path.exists(binding.LIB_PATH), "libsurel.so is not built"
    c = binding.Context()
    yield c
    c.close()


def dev(a, dtype=None):
    t = torch.from_numpy(np.ascontiguousarray(a))
    if dtype is not None:
        t = t.to(dtype)
    return t.cuda()


def host_u16(t):
    return t.view(torch.int16).cpu().numpy().view(np.uint16)


def gpu_pipeline(ctx, rp, ci, seeds, M, m, rng_seed, queries=None, with_sizes=False):
    """walks -> RPE -> join on the GPU.  ``with_sizes``: the walk kernel reports |V_u| and
    build_rpe lays the table out from that; otherwise build_rpe counts by itself."""
    d_rp, d_ci, d_seeds = dev(rp), dev(ci), dev(np.asarray(seeds, dtype=np.int32))
    n_nodes = rp.size - 1
    sizes = None
    if with_sizes:
        sizes = torch.full((d_seeds.numel(),), -1, dtype=torch.int32, device="cuda")
    walks = binding.sample_walks(ctx, d_rp, d_ci, d_seeds, M, m, rng_seed, set_sizes=sizes)
    off, ids, cnt = binding.build_rpe(ctx, walks, n_nodes, set_sizes=sizes)
    out = {"walks": walks, "rpe": (off, ids, cnt), "sizes": sizes}
    if queries is not None:
        d_q = dev(np.asarray(queries, dtype=np.int32))
        out["join"] = binding.join_queries(ctx, off, ids, cnt, d_q, max_set=1 + M * m)
    assert ctx.check() == 0
    return out


def assert_table_equal(got, want, what):
    g_off, g_ids, g_cnt = got
    w_off, w_ids, w_cnt = want
    assert np.array_equal(g_off.cpu().numpy(), w_off), f"{what}: offsets differ"
    assert np.array_equal(g_ids.cpu().numpy(), w_ids), f"{what}: ids differ"
    assert np.array_equal(host_u16(g_cnt), w_cnt), f"{what}: counts differ"


def full_compare(ctx, rp, ci, seeds, M, m, rng_seed, queries):
    w = oracle.sample_walks(rp, ci, seeds, M, m, rng_seed)
    table = oracle.build_rpe(w)
    joined = oracle.join_queries(*table, queries) if queries is not None else None
    for with_sizes in (False, True):
        out = gpu_pipeline(ctx, rp, ci, seeds, M, m, rng_seed, queries, with_sizes)
        assert np.array_equal(out["walks"].cpu().numpy(), w), "walks differ"
        if with_sizes:
            assert np.array_equal(out["sizes"].cpu().numpy(), np.diff(table[0])), "set sizes"
        assert_table_equal(out["rpe"], table, f"rpe (sizes from walks: {with_sizes})")
        if queries is not None:
            assert_table_equal(out["join"], joined, "join")
    # the fused walk + RPE kernel gives the same walks and the same table
    d_seeds = dev(np.asarray(seeds, dtype=np.int32))
    f_walks, f_off, f_ids, f_cnt = binding.sample_walks_rpe(ctx, dev(rp), dev(ci), d_seeds, M, m,
                                                            rng_seed)
    assert ctx.check() == 0
    assert np.array_equal(f_walks.cpu().numpy(), w), "fused: walks differ"
    assert_table_equal((f_off, f_ids, f_cnt), table, "fused rpe")
    # the pruned central array and the re-indexed rows
    T, code = binding.prune_rpe(ctx, f_cnt, cap_T=max(1, table[2].shape[0]))
    assert ctx.check() == 0
    want_T, want_code = oracle.prune_rpe(table[2])
    assert np.array_equal(host_u16(T), want_T), "pruned array differs"
    assert np.array_equal(code.cpu().numpy(), want_code), "re-indexed rows differ"
    # walks, table and pruned array from one call, with and without the count vectors
    for with_counts in (True, False):
        i_walks, i_off, i_ids, i_cnt, i_code, i_T = binding.sample_walks_rpe_ids(
            ctx, dev(rp), dev(ci), d_seeds, M, m, rng_seed, cap_T=max(1, table[2].shape[0]),
            with_counts=with_counts)
        assert ctx.check() == 0
        assert np.array_equal(i_walks.cpu().numpy(), w), "one call: walks differ"
        assert np.array_equal(i_off.cpu().numpy(), table[0]), "one call: offsets differ"
        assert np.array_equal(i_ids.cpu().numpy(), table[1]), "one call: ids differ"
        if with_counts:
            assert np.array_equal(host_u16(i_cnt), table[2]), "one call: counts differ"
        assert np.array_equal(host_u16(i_T).reshape(want_T.shape), want_T), "one call: T differs"
        assert np.array_equal(i_code.cpu().numpy(), want_code), "one call: codes differ"
    if queries is not None and np.asarray(queries).shape[0] > 0:
        # query-level RPE-IDs of every walk position
        got = binding.query_rpe_ids(ctx, f_walks, f_off, f_ids, dev(np.asarray(queries, np.int32)),
                                    max_set=1 + M * m)
        assert ctx.check() == 0
        want = oracle.query_rpe_ids(w, table[0], table[1], queries)
        assert np.array_equal(got.cpu().numpy().astype(np.int64), want), "query RPE-IDs differ"
        # the same as indices into the pruned array: the code of the row, -1 where there is none
        got = binding.query_rpe_ids(ctx, f_walks, f_off, f_ids, dev(np.asarray(queries, np.int32)),
                                    max_set=1 + M * m, code=code)
        assert ctx.check() == 0
        want_ids = np.where(want < 0, -1, want_code.astype(np.int64)[np.maximum(want, 0)])
        assert np.array_equal(got.cpu().numpy().astype(np.int64), want_ids), "pruned RPE-IDs differ"
        # the union join over the codes: the same rows, every count vector replaced by its index
        # in the oracle's pruned array (-1 for the all-zero vector of an absent node)
        j_off, j_ids, j_codes = binding.join_query_ids(ctx, f_off, f_ids, code,
                                                       dev(np.asarray(queries, np.int32)),
                                                       max_set=1 + M * m)
        assert ctx.check() == 0
        index_of = {tuple(v): i for i, v in enumerate(want_T.tolist())}
        want_codes = np.array([[index_of.get(tuple(vec), -1) if any(vec) else -1 for vec in row]
                               for row in joined[2].tolist()], dtype=np.int32).reshape(-1, len(queries[0]))
        assert np.array_equal(j_off.cpu().numpy(), joined[0]), "join offsets differ (ids form)"
        assert np.array_equal(j_ids.cpu().numpy(), joined[1]), "join ids differ (ids form)"
        assert np.array_equal(j_codes.cpu().numpy(), want_codes), "joined RPE-IDs differ"
    return out


# --------------------------------------------------------------------------- #
# small and medium inputs, element by element
# --------------------------------------------------------------------------- #
def test_tensor_arguments_give_their_addresses(ctx):
    t = torch.arange(40, dtype=torch.int32, device="cuda")
    u16 = t.to(torch.int16).view(torch.uint16)
    for x in (t, t[3:], t.view(8, 5)[2:], t[:0], u16, u16[1:], torch.nn.Parameter(t.float())):
        assert binding._ptr(x, x.dtype, "x") == binding._ptr_in_python(x, x.dtype, "x") == x.data_ptr()
    for x in (t.view(8, 5).t(), t[::2]):
        with pytest.raises(ValueError, match="contiguous"):
            binding._ptr(x, torch.int32, "x")
    with pytest.raises(TypeError, match="x must be torch.int64, got torch.int32"):
        binding._ptr(t, torch.int64, "x")


def test_rmat4k_whole_pipeline_bit_exact(ctx):
    wl = synth.WORKLOADS["rmat4k"]
    rp, ci = synth.make_graph(wl)
    queries = synth.make_queries(wl, rp, ci)
    seeds = np.arange(wl.n_nodes, dtype=np.int32)
    full_compare(ctx, rp, ci, seeds, wl.M, wl.m, wl.rng_seed, queries)


@pytest.mark.parametrize("M,m", [(1, 1), (3, 2), (50, 4), (64, 3), (65, 3), (100, 4), (130, 3),
                                 (200, 4), (200, 3), (128, 15), (400, 4), (341, 5), (7, 15)])
@pytest.mark.parametrize("k", [2, 3])
def test_shapes_bit_exact(ctx, M, m, k):
    wl = synth.Workload("t", "rmat", 1024, 5000, 0.0, M, m, 300, k, "uniform",
                        graph_seed=100 + M + m)
    rp, ci = synth.make_graph(wl)
    rng = np.random.default_rng(M * 31 + m)
    # a ragged, unordered seed list with repeats: 4 waves per workgroup leave a tail
    seeds = rng.integers(0, wl.n_nodes, size=203).astype(np.int32)
    queries = rng.integers(0, seeds.size, size=(301, k)).astype(np.int32)
    queries[0] = 5                                    # every entry the same block
    full_compare(ctx, rp, ci, seeds, M, m, 0xABCDEF0123456789 & ((1 << 64) - 1), queries)


def test_tiny_graphs_and_isolated_nodes(ctx):
    # path 0-1-2-3, isolated node 4, star centred on 5 with leaves 6..9
    rp, ci = synth.csr_from_edge_list(10, [(0, 1), (1, 2), (2, 3), (5, 6), (5, 7), (5, 8), (5, 9)])
    seeds = np.arange(10, dtype=np.int32)
    queries = np.array([[4, 4], [4, 0], [0, 3], [5, 6], [9, 4]], dtype=np.int32)
    out = full_compare(ctx, rp, ci, seeds, 33, 4, 7, queries)
    walks = out["walks"].cpu().numpy()
    assert (walks[4] == 4).all()
    assert (walks[0, :, 1] == 1).all()


def test_edgeless_graph(ctx):
    rp = np.zeros(6, dtype=np.int32)
    ci = np.zeros(0, dtype=np.int32)
    seeds = np.array([3, 0, 4], dtype=np.int32)
    queries = np.array([[0, 1], [2, 2]], dtype=np.int32)
    full_compare(ctx, rp, ci, seeds, 10, 3, 1, queries)


def test_empty_seed_and_query_lists(ctx):
    wl = synth.WORKLOADS["rmat4k"]
    rp, ci = synth.make_graph(wl)
    out = gpu_pipeline(ctx, rp, ci, np.zeros(0, dtype=np.int32), 50, 4, 0,
                       np.zeros((0, 2), dtype=np.int32))
    assert out["walks"].shape == (0, 50, 5)
    off, ids, cnt = out["rpe"]
    assert off.cpu().tolist() == [0] and ids.numel() == 0 and cnt.numel() == 0
    joff, jids, jcnt = out["join"]
    assert joff.cpu().tolist() == [0] and jids.numel() == 0
    # an empty query list against a non-empty table
    out = gpu_pipeline(ctx, rp, ci, np.arange(8, dtype=np.int32), 50, 4, 0,
                       np.zeros((0, 3), dtype=np.int32))
    assert out["join"][0].cpu().tolist() == [0]


def test_paper_worked_example_on_the_gpu(ctx, golden_dir):
    from test_oracle_pins import _read_example
    ex = _read_example(golden_dir)
    m, M = ex["m"][0], ex["M"][0]
    walks = np.array([ex["walks_u"], ex["walks_v"]], dtype=np.int32).reshape(2, M, m + 1)
    off, ids, cnt = binding.build_rpe(ctx, dev(walks), n_nodes=7)
    joff, jids, jcnt = binding.join_queries(ctx, off, ids, cnt, dev(np.array([[0, 1]], np.int32)),
                                            max_set=1 + M * m)
    assert ctx.check() == 0
    ids_h, cnt_h = ids.cpu().numpy(), host_u16(cnt)
    blk = slice(int(off[0]), int(off[1]))
    assert cnt_h[blk][ids_h[blk] == 0][0].tolist() == ex["X_u,u"]
    assert cnt_h[blk][ids_h[blk] == 2][0].tolist() == ex["X_u,a"]
    assert cnt_h[blk][ids_h[blk] == 1][0].tolist() == ex["X_u,v"]
    row = host_u16(jcnt)[jids.cpu().numpy() == 0][0]
    assert row.reshape(-1).tolist() == ex["X_Q,u"]
    assert_table_equal((off, ids, cnt), oracle.build_rpe(walks), "rpe")


def test_hand_made_walks_with_mixed_start_nodes(ctx):
    # build_rpe counts whatever the walk block holds, also when position 0 varies
    rng = np.random.default_rng(4)
    walks = rng.integers(0, 40, size=(37, 20, 4)).astype(np.int32)
    off, ids, cnt = binding.build_rpe(ctx, dev(walks), n_nodes=40)
    assert ctx.check() == 0
    assert_table_equal((off, ids, cnt), oracle.build_rpe(walks), "rpe")


def test_two_runs_are_identical(ctx):
    wl = synth.WORKLOADS["rmat4k"]
    rp, ci = synth.make_graph(wl)
    queries = synth.make_queries(wl, rp, ci)
    seeds = np.arange(wl.n_nodes, dtype=np.int32)
    a = gpu_pipeline(ctx, rp, ci, seeds, wl.M, wl.m, 5, queries)
    b = gpu_pipeline(ctx, rp, ci, seeds, wl.M, wl.m, 5, queries)
    assert torch.equal(a["walks"], b["walks"])
    for x, y in zip(a["rpe"] + a["join"], b["rpe"] + b["join"]):
        assert torch.equal(x.view(torch.int16) if x.dtype == torch.uint16 else x,
                           y.view(torch.int16) if y.dtype == torch.uint16 else y)


# --------------------------------------------------------------------------- #
# device-detected problems never fault and are reported
# --------------------------------------------------------------------------- #
def test_bad_seed_is_flagged_and_skipped(ctx):
    rp, ci = synth.csr_from_edge_list(5, [(0, 1), (1, 2), (2, 3), (3, 4)])
    seeds = np.array([1, 99, -3, 2], dtype=np.int32)
    walks = binding.sample_walks(ctx, dev(rp), dev(ci), dev(seeds), 9, 3, 0)
    assert ctx.check() == binding.DEV_BAD_SEED
    assert ctx.check() == 0                                # the word is cleared by the read
    w = walks.cpu().numpy()
    assert (w[1] == -1).all() and (w[2] == -1).all()
    good = oracle.sample_walks(rp, ci, seeds[[0, 3]], 9, 3, 0)
    assert np.array_equal(w[[0, 3]], good)


def test_malformed_csr_is_flagged(ctx):
    rp = np.array([0, 2, 4, 6], dtype=np.int32)
    ci = np.array([1, 2, 0, 77, 0, 1], dtype=np.int32)     # node 77 does not exist
    walks = binding.sample_walks(ctx, dev(rp), dev(ci), dev(np.arange(3, dtype=np.int32)), 64, 4, 0)
    assert ctx.check() == binding.DEV_BAD_GRAPH
    w = walks.cpu().numpy()
    assert ((w >= 0) & (w < 3)).all()


def test_bad_walk_entry_is_flagged(ctx):
    walks = np.zeros((3, 4, 3), dtype=np.int32)
    walks[1, 2, 1] = 1000
    off = torch.empty(4, dtype=torch.int64, device="cuda")
    rc, rows = binding.build_rpe_raw(ctx, dev(walks), 10, 0, off, None, None)
    assert rc == binding.OK and rows == 3
    assert ctx.check() == binding.DEV_BAD_WALK


def test_wrong_set_sizes_are_flagged_and_do_not_overlap(ctx):
    wl = synth.Workload("t", "rmat", 256, 900, 0.0, 20, 3, 0, 2, "uniform", graph_seed=3)
    rp, ci = synth.make_graph(wl)
    seeds = np.arange(16, dtype=np.int32)
    sizes = torch.empty(16, dtype=torch.int32, device="cuda")
    walks = binding.sample_walks(ctx, dev(rp), dev(ci), dev(seeds), wl.M, wl.m, 0, set_sizes=sizes)
    want_off, want_ids, want_cnt = oracle.build_rpe(walks.cpu().numpy())
    sizes[5] += 3                                         # a size that is not this seed's
    total = int(want_off[-1]) + 3
    off = torch.empty(17, dtype=torch.int64, device="cuda")
    ids = torch.full((total,), -7, dtype=torch.int32, device="cuda")
    cnt = torch.zeros((total, wl.m + 1), dtype=torch.int16, device="cuda").view(torch.uint16)
    rc, rows = binding.build_rpe_raw(ctx, walks, wl.n_nodes, total, off, ids, cnt,
                                     set_sizes=sizes)
    assert rc == binding.OK and rows == total
    assert ctx.check() == binding.DEV_BAD_SIZES
    ids_h = ids.cpu().numpy()
    lo, hi = int(want_off[5]), int(want_off[6]) + 3
    assert (ids_h[lo:hi] == -7).all()                      # the mismatched seed wrote nothing
    assert np.array_equal(ids_h[:lo], want_ids[:lo])       # the others are where sizes put them
    assert np.array_equal(ids_h[hi:], want_ids[int(want_off[6]):])


def test_rpe_capacity_overflow_is_reported_and_nothing_is_written_past_it(ctx):
    wl = synth.Workload("t", "rmat", 256, 900, 0.0, 20, 3, 0, 2, "uniform", graph_seed=3)
    rp, ci = synth.make_graph(wl)
    seeds = np.arange(64, dtype=np.int32)
    walks = binding.sample_walks(ctx, dev(rp), dev(ci), dev(seeds), wl.M, wl.m, 0)
    want_off, want_ids, want_cnt = oracle.build_rpe(walks.cpu().numpy())
    total = int(want_off[-1])
    cap = total // 2
    L = wl.m + 1
    off = torch.empty(65, dtype=torch.int64, device="cuda")
    ids = torch.full((total,), -7, dtype=torch.int32, device="cuda")
    cnt = torch.full((total, L), 0x7777, dtype=torch.int16, device="cuda").view(torch.uint16)
    rc, rows = binding.build_rpe_raw(ctx, walks, wl.n_nodes, cap, off, ids, cnt)
    assert rc == binding.E_CAPACITY and rows == total
    assert ctx.check() == binding.DEV_CAPACITY
    assert np.array_equal(off.cpu().numpy(), want_off)      # offsets are complete anyway
    ids_h, cnt_h = ids.cpu().numpy(), host_u16(cnt)
    assert (ids_h[cap:] == -7).all() and (cnt_h[cap:] == 0x7777).all()
    fits = want_off[1:] <= cap                               # blocks that fit are written
    last = int(want_off[1:][fits].max())
    assert np.array_equal(ids_h[:last], want_ids[:last])
    assert np.array_equal(cnt_h[:last], want_cnt[:last])


@pytest.mark.parametrize("n_seeds", [64, 6000])
def test_fused_bad_seed_capacity_and_count_only(ctx, n_seeds):
    # 64 seeds take one launch without roles, 6,000 the persistent kernel
    wl = synth.Workload("t", "rmat", 256, 900, 0.0, 20, 3, 0, 2, "uniform", graph_seed=3)
    rp, ci = synth.make_graph(wl)
    M, m, L = wl.M, wl.m, wl.m + 1
    seeds = np.arange(n_seeds, dtype=np.int32) % wl.n_nodes
    bad = [7, 20] + ([4500, n_seeds - 1] if n_seeds > 4500 else [])
    seeds[bad] = ([1000, -1] * 2)[:len(bad)]                 # not nodes
    good = np.ones(n_seeds, dtype=bool)
    good[bad] = False
    w = oracle.sample_walks(rp, ci, seeds[good], M, m, 3)
    want_off, want_ids, want_cnt = oracle.build_rpe(w)
    sizes = np.zeros(n_seeds, dtype=np.int64)
    sizes[good] = np.diff(want_off)
    full_off = np.concatenate([[0], np.cumsum(sizes)])
    total = int(full_off[-1])
    d_rp, d_ci, d_seeds = dev(rp), dev(ci), dev(seeds)
    walks = torch.empty((n_seeds, M, L), dtype=torch.int32, device="cuda")
    off = torch.empty(n_seeds + 1, dtype=torch.int64, device="cuda")
    # offsets and total only
    rc, rows = binding.sample_walks_rpe_raw(ctx, d_rp, d_ci, d_seeds, M, m, 3, walks, 0, off,
                                            None, None)
    assert rc == binding.OK and rows == total
    assert ctx.check() == binding.DEV_BAD_SEED
    assert np.array_equal(off.cpu().numpy(), full_off)
    wh = walks.cpu().numpy()
    assert (wh[bad] == -1).all() and np.array_equal(wh[good], w)
    # a table that is too small: complete offsets, nothing written at or past cap_rows
    cap = total // 2
    ids = torch.full((total,), -7, dtype=torch.int32, device="cuda")
    cnt = torch.full((total, L), 0x7777, dtype=torch.int16, device="cuda").view(torch.uint16)
    rc, rows = binding.sample_walks_rpe_raw(ctx, d_rp, d_ci, d_seeds, M, m, 3, walks, cap, off,
                                            ids, cnt)
    assert rc == binding.E_CAPACITY and rows == total
    assert ctx.check() == binding.DEV_BAD_SEED | binding.DEV_CAPACITY
    assert np.array_equal(off.cpu().numpy(), full_off)
    ids_h, cnt_h = ids.cpu().numpy(), host_u16(cnt)
    assert (ids_h[cap:] == -7).all() and (cnt_h[cap:] == 0x7777).all()
    last = int(full_off[1:][full_off[1:] <= cap].max())
    assert np.array_equal(ids_h[:last], want_ids[:last])
    assert np.array_equal(cnt_h[:last], want_cnt[:last])
    # no seeds at all
    rc, rows = binding.sample_walks_rpe_raw(ctx, d_rp, d_ci, d_seeds[:0], M, m, 3, walks[:0], 0,
                                            off[:1], None, None)
    assert rc == binding.OK and rows == 0 and int(off[0]) == 0


@pytest.mark.parametrize("M,m", [(50, 4), (200, 3)])
def test_fused_kernel_seed_counts_around_its_group_and_window_sizes(ctx, M, m):
    # seeds are handed out in groups of 8 and the offset scan reads 2048 counts a round: seed
    # counts on, just below and just above those sizes, against the two-call path
    wl = synth.Workload("t", "rmat", 2048, 12000, 0.0, M, m, 0, 2, "uniform", graph_seed=5)
    rp, ci = synth.make_graph(wl)
    d_rp, d_ci = dev(rp), dev(ci)
    rng = np.random.default_rng(8)
    all_seeds = dev(rng.integers(0, wl.n_nodes, size=20000).astype(np.int32))
    for n in (1, 2, 7, 8, 9, 15, 16, 17, 63, 64, 65, 511, 2047, 2048, 2049, 4104, 16384, 16391,
              20000):
        d_seeds = all_seeds[:n].contiguous()
        walks = binding.sample_walks(ctx, d_rp, d_ci, d_seeds, M, m, 11)
        off, ids, cnt = binding.build_rpe(ctx, walks, wl.n_nodes)
        f_walks, f_off, f_ids, f_cnt = binding.sample_walks_rpe(ctx, d_rp, d_ci, d_seeds, M, m, 11)
        assert ctx.check() == 0
        assert torch.equal(f_walks, walks), f"walks differ at {n} seeds"
        assert torch.equal(f_off, off), f"offsets differ at {n} seeds"
        assert torch.equal(f_ids, ids), f"ids differ at {n} seeds"
        assert torch.equal(f_cnt.view(torch.int16), cnt.view(torch.int16)), f"counts differ at {n}"


@pytest.mark.parametrize("n_seeds,n_queries", [(1500, 700), (6000, 5000)])
def test_one_pass_captured_in_a_graph_replays_to_the_same_bytes(n_seeds, n_queries):
    # with no row totals asked for, the calls only enqueue kernels: a pass can be captured once
    # and replayed; every replay (with other work on the stream in between) gives the eager bytes.
    # Few seeds and queries take one launch each, more take the persistent kernel and two launches
    wl = synth.Workload("t", "rmat", 4096, 30000, 0.0, 50, 4, 0, 2, "uniform", graph_seed=9)
    rp, ci = synth.make_graph(wl)
    rng = np.random.default_rng(4)
    seeds = rng.integers(0, wl.n_nodes, size=n_seeds).astype(np.int32)
    queries = rng.integers(0, seeds.size, size=(n_queries, 2)).astype(np.int32)
    M, m, L, S = wl.M, wl.m, wl.m + 1, seeds.size
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        c = binding.Context(stream=stream)
        d_rp, d_ci, d_seeds, d_q = dev(rp), dev(ci), dev(seeds), dev(queries)
        cap_r = binding.rpe_rows_bound(S, M, m)
        walks = torch.empty((S, M, L), dtype=torch.int32, device="cuda")
        off = torch.empty(S + 1, dtype=torch.int64, device="cuda")
        ids = torch.empty(cap_r, dtype=torch.int32, device="cuda")
        cnt = torch.empty((cap_r, L), dtype=torch.uint16, device="cuda")
        joff = torch.empty(queries.shape[0] + 1, dtype=torch.int64, device="cuda")
        max_set = 1 + M * m
        # eager pass: sizes the join's output, warms the context's workspaces, is the reference
        rc, R = binding.sample_walks_rpe_raw(c, d_rp, d_ci, d_seeds, M, m, 5, walks, cap_r, off, ids, cnt)
        assert rc == binding.OK
        rc, J = binding.join_queries_raw(c, off, ids, cnt, d_q, max_set, 0, joff, None, None)
        assert rc == binding.OK
        jids = torch.empty(J, dtype=torch.int32, device="cuda")
        jcnt = torch.empty((J, 2, L), dtype=torch.uint16, device="cuda")
        rc, _ = binding.join_queries_raw(c, off, ids, cnt, d_q, max_set, J, joff, jids, jcnt)
        assert rc == binding.OK and c.check() == 0
        outs = [walks, off, ids[:R], cnt[:R].view(torch.int16), joff, jids, jcnt.view(torch.int16)]
        want = [t.clone() for t in outs]

        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream, capture_error_mode="thread_local"):
            rc1, _ = binding.sample_walks_rpe_raw(c, d_rp, d_ci, d_seeds, M, m, 5, walks, cap_r, off,
                                                  ids, cnt, want_rows=False)
            rc2, _ = binding.join_queries_raw(c, off, ids, cnt, d_q, max_set, J, joff, jids, jcnt,
                                              want_rows=False)
        assert rc1 == binding.OK and rc2 == binding.OK
        for replay in range(3):
            for t in outs:
                t.fill_(-7 - replay)                 # eager work between the replays
            stream.synchronize()
            graph.replay()
            stream.synchronize()
            assert c.check() == 0, f"replay {replay}"
            for got, ref in zip(outs, want):
                assert torch.equal(got, ref), f"replay {replay} differs from the eager pass"
        c.close()


@pytest.mark.parametrize("M,m", [(1, 1), (21, 2), (32, 1), (16, 3), (13, 4), (22, 2), (33, 1)])
def test_blocks_of_about_one_value_a_lane(ctx, M, m):
    # walk blocks of 2, 63, 64, 65 and 66 values and the rows of as many nodes, in outputs that start
    # anywhere inside 16 bytes, from the fused kernel and from the separate calls
    rng = np.random.default_rng(M)
    n, L = 9000, m + 1
    rp = (np.arange(n + 1) * 40).astype(np.int32)
    ci = rng.integers(0, n, size=40 * n).astype(np.int32)
    seeds = rng.integers(0, n, size=n).astype(np.int32)
    want = oracle.sample_walks(rp, ci, seeds, M, m, 5)
    table = oracle.build_rpe(want)
    R, d_rp, d_ci, d_seeds = table[1].size, dev(rp), dev(ci), dev(seeds)
    for skip in (0, 2, 4, 6) if L % 2 else (0, 1, 2, 3):  # count vectors start at aligned words
        walks = torch.full((n * M * L + 8,), -7, dtype=torch.int32, device="cuda")
        ids = torch.full((R + 8,), -7, dtype=torch.int32, device="cuda")
        cnt = torch.full((R + 8, L), 9, dtype=torch.int16, device="cuda").view(torch.uint16)
        off = torch.empty(n + 1, dtype=torch.int64, device="cuda")
        w = walks[skip:skip + n * M * L].view(n, M, L)
        rc, rows = binding.sample_walks_rpe_raw(ctx, d_rp, d_ci, d_seeds, M, m, 5, w, R, off,
                                                ids[skip:skip + R], cnt[skip:skip + R])
        assert rc == binding.OK and rows == R and ctx.check() == 0
        assert np.array_equal(w.cpu().numpy(), want)
        assert_table_equal((off, ids[skip:skip + R], cnt[skip:skip + R]), table, f"fused, from {skip}")
        ids[skip:skip + R], cnt.view(torch.int16)[skip:skip + R] = -7, 9
        rc, rows = binding.build_rpe_raw(ctx, w, n, R, off, ids[skip:skip + R], cnt[skip:skip + R])
        assert rc == binding.OK and rows == R and ctx.check() == 0
        assert_table_equal((off, ids[skip:skip + R], cnt[skip:skip + R]), table, f"table, from {skip}")
        for rest, whole in ((-7, walks), (-7, ids), (9, cnt.view(torch.int16))):
            size = whole.shape[0] - 8
            assert (whole[:skip] == rest).all() and (whole[skip + size:] == rest).all()


def test_fused_kernel_waits_are_bounded(ctx):
    # with a spin limit of zero every wait inside the fused kernel gives up at once: the kernel
    # must still end, say so, and write nothing out of place; the default limit then gives the
    # right table again
    wl = synth.Workload("t", "rmat", 4096, 30000, 0.0, 50, 4, 0, 2, "uniform", graph_seed=9)
    rp, ci = synth.make_graph(wl)
    seeds = np.arange(wl.n_nodes, dtype=np.int32)
    d_rp, d_ci, d_seeds = dev(rp), dev(ci), dev(seeds)
    M, m, L = wl.M, wl.m, wl.m + 1
    cap = binding.rpe_rows_bound(seeds.size, M, m)
    walks = torch.empty((seeds.size, M, L), dtype=torch.int32, device="cuda")
    off = torch.empty(seeds.size + 1, dtype=torch.int64, device="cuda")
    ids = torch.full((cap,), -7, dtype=torch.int32, device="cuda")
    cnt = torch.zeros((cap, L), dtype=torch.int16, device="cuda").view(torch.uint16)
    ctx.set_spin_limit(0)
    try:
        rc, _ = binding.sample_walks_rpe_raw(ctx, d_rp, d_ci, d_seeds, M, m, 0, walks, cap, off,
                                             ids, cnt, want_rows=False)
        assert rc == binding.OK
        flags = ctx.check()
    finally:
        ctx.set_spin_limit(1 << 22)
    assert flags & ~binding.DEV_STALL == 0
    w = oracle.sample_walks(rp, ci, seeds, M, m, 0)
    want = oracle.build_rpe(w)
    if flags == 0:
        assert_table_equal((off, ids[:int(off[-1])], cnt[:int(off[-1])]), want, "rpe")
    else:
        # whatever was written is a correct prefix of the table or untouched memory
        ids_h = ids.cpu().numpy()[:want[1].size]
        assert ((ids_h == want[1]) | (ids_h == -7)).all()
    f_walks, f_off, f_ids, f_cnt = binding.sample_walks_rpe(ctx, d_rp, d_ci, d_seeds, M, m, 0)
    assert ctx.check() == 0
    assert np.array_equal(f_walks.cpu().numpy(), w)
    assert_table_equal((f_off, f_ids, f_cnt), want, "rpe after the limit was restored")


@pytest.mark.parametrize("spins", [0, 2, 4, 6, 8, 10, 12, 16, 24])
def test_a_wait_that_runs_out_in_the_fused_kernel_is_reported(ctx, spins):
    # more seeds than go into one launch without roles; whichever wave gives up (the scanner, or a
    # worker whose counts the scanner has), a call that was given h_rows says so
    wl = synth.Workload("t", "rmat", 16384, 100000, 0.0, 50, 4, 0, 2, "uniform", graph_seed=9)
    rp, ci = synth.make_graph(wl)
    seeds = np.arange(wl.n_nodes, dtype=np.int32)
    d_rp, d_ci, d_seeds = dev(rp), dev(ci), dev(seeds)
    M, m, L = wl.M, wl.m, wl.m + 1
    want = binding.sample_walks_rpe(ctx, d_rp, d_ci, d_seeds, M, m, 1)
    want_T, want_code = binding.prune_rpe(ctx, want[3], cap_T=4096)
    assert ctx.check() == 0
    cap = want[2].numel()
    walks = torch.empty((seeds.size, M, L), dtype=torch.int32, device="cuda")
    off = torch.empty(seeds.size + 1, dtype=torch.int64, device="cuda")
    ids, code = (torch.empty(cap, dtype=torch.int32, device="cuda") for _ in range(2))
    cnt = torch.empty((cap, L), dtype=torch.uint16, device="cuda")
    T = torch.zeros((4096, L), dtype=torch.int16, device="cuda").view(torch.uint16)
    for with_ids in (False, True):
        ids.fill_(-7)
        ctx.set_spin_limit(spins)
        try:
            if with_ids:
                rc, rows, n_T = binding.sample_walks_rpe_ids_raw(ctx, d_rp, d_ci, d_seeds, M, m, 1, walks,
                                                                 cap, off, ids, None, code, 4096, T)
            else:
                rc, rows = binding.sample_walks_rpe_raw(ctx, d_rp, d_ci, d_seeds, M, m, 1, walks, cap,
                                                        off, ids, cnt)
        finally:
            ctx.set_spin_limit(1 << 22)
        flags = ctx.check()
        print(f"spins {spins} ids {with_ids}: status {rc}, flags {flags:#x}", flush=True)
        if rc == binding.OK:
            assert flags == 0 and rows == cap
            assert torch.equal(off, want[1]) and torch.equal(ids, want[2])
            if with_ids:
                assert n_T == want_T.shape[0] and torch.equal(code, want_code)
        else:
            assert rc == binding.E_DEVICE and flags == binding.DEV_STALL and rows == -1
    # the next call is right again, its hash set is what it should be
    rc, rows, n_T = binding.sample_walks_rpe_ids_raw(ctx, d_rp, d_ci, d_seeds, M, m, 1, walks, cap, off,
                                                     ids, None, code, 4096, T)
    assert rc == binding.OK and rows == cap and ctx.check() == 0
    assert torch.equal(ids, want[2]) and torch.equal(code, want_code)


def test_prune_capacity_and_degenerate_tables(ctx):
    rng = np.random.default_rng(3)
    cnt = rng.integers(0, 3, size=(5000, 4)).astype(np.uint16)          # at most 81 vectors
    want_T, want_code = oracle.prune_rpe(cnt)
    d_cnt = dev(cnt.view(np.int16)).view(torch.uint16)
    n_T = want_T.shape[0]
    T = torch.zeros((n_T, 4), dtype=torch.int16, device="cuda").view(torch.uint16)
    code = torch.empty(5000, dtype=torch.int32, device="cuda")
    rc, got = binding.prune_rpe_raw(ctx, d_cnt, n_T, T, code)           # exactly enough room
    assert rc == binding.OK and got == n_T and ctx.check() == 0
    assert np.array_equal(host_u16(T), want_T) and np.array_equal(code.cpu().numpy(), want_code)
    rc, got = binding.prune_rpe_raw(ctx, d_cnt, n_T - 1, T, code)       # one too few
    assert rc == binding.E_CAPACITY and got == n_T
    assert ctx.check() == binding.DEV_CAPACITY
    # one row, all rows equal, widest vectors (m = 15), no rows
    for arr in (np.array([[7, 0, 9]], np.uint16), np.full((300, 5), 65535, np.uint16),
                rng.integers(0, 2, size=(700, 16)).astype(np.uint16),
                np.zeros((0, 4), np.uint16)):
        T, code = binding.prune_rpe(ctx, dev(arr.view(np.int16)).view(torch.uint16), cap_T=1024)
        assert ctx.check() == 0
        w_T, w_code = oracle.prune_rpe(arr)
        assert np.array_equal(host_u16(T).reshape(w_T.shape), w_T)
        assert np.array_equal(code.cpu().numpy(), w_code)


@pytest.mark.parametrize("L,n_T", [(2, 70_710), (2, 70_711), (5, 40_824), (5, 40_825), (16, 25_000),
                                   (16, 25_001), (16, 1 << 15), (9, 100_003)])
def test_prune_of_many_distinct_vectors(ctx, L, n_T):
    # on both sides of the line from which the vectors are sorted instead of compared all with all,
    # a list that needs no padding, and more than the codes of 16 bits could tell apart; vectors
    # occur once, twice or often, neighbours in a wave are mostly different
    rng = np.random.default_rng(n_T)
    vectors = rng.integers(0, 4, size=(n_T, L)).astype(np.uint16)
    number = rng.permutation(n_T)
    vectors[:, 0], vectors[:, -1] = number % 400, number // 400
    rows = np.concatenate([np.arange(n_T), rng.integers(0, n_T, size=n_T // 2),
                           rng.integers(0, 50, size=3001)])
    cnt = vectors[rng.permutation(rows)]
    want_T, want_code = oracle.prune_rpe(cnt)
    assert want_T.shape[0] == n_T
    d_cnt = dev(cnt.view(np.int16)).view(torch.uint16)
    for cap_T in (n_T, 1 << 18):
        T, code = binding.prune_rpe(ctx, d_cnt, cap_T=cap_T)
        assert ctx.check() == 0
        assert np.array_equal(host_u16(T), want_T) and np.array_equal(code.cpu().numpy(), want_code)


@pytest.mark.parametrize("L", [2, 3, 5, 6, 10])
@pytest.mark.parametrize("n_rows,n_T,most", [(1, 1, 3), (127, 9, 3), (512, 512, 200), (513, 40, 3),
                                             (3_000_003, 300, 7), (3_000_003, 1500, 90),
                                             (2_200_000, 40_000, 300), (1 << 25, 1500, 90),
                                             ((1 << 25) + 1, 1500, 90), ((1 << 25) + 513, 40_000, 300)])
def test_prune_lists_of_rows_that_wait_for_a_look_up(ctx, L, n_rows, n_T, most):
    # around a tile of 512 rows and the rows looked up first; tables whose rows the direct table knows,
    # the hashed cache knows, or neither, so that the list of late rows fills, is emptied over several
    # tiles, and has no room; few rows and many (more than 2^25): T is sorted and distinct, and every row's
    # code names its vector
    g = torch.Generator(device="cuda").manual_seed(n_rows + L)
    vectors = torch.randint(0, most + 1, (4 * n_T, L), device="cuda", generator=g)
    vectors[::2, 0] = 0
    vectors = torch.unique(vectors, dim=0)
    vectors = vectors[torch.randperm(vectors.shape[0], device="cuda", generator=g)[:n_T]]
    # common ones and rare ones
    pick = (torch.rand(n_rows, device="cuda", generator=g) ** 3 * vectors.shape[0]).long()
    cnt = vectors[pick].to(torch.int16).contiguous().view(torch.uint16)
    T, code = binding.prune_rpe(ctx, cnt, cap_T=1 << 18)
    assert ctx.check() == 0
    want = torch.unique(vectors[torch.unique(pick)], dim=0)  # sorted entry by entry
    assert torch.equal(T.view(torch.int16).long(), want)
    assert torch.equal(T.view(torch.int16)[code.long()], cnt.view(torch.int16))


@pytest.mark.parametrize("M,m", [(149, 3), (112, 4), (112, 3), (115, 5), (144, 4), (144, 3), (277, 3),
                                 (208, 4), (208, 3), (179, 5), (224, 4), (224, 3)])
def test_sorts_of_odd_numbers_of_keys_a_lane(ctx, M, m):
    # the last number of keys of a sort and the first of the next one, for 7, 9, 13 and 14 keys a lane, of
    # M*m + 1 keys (walks + RPE, for many seeds and for few) and of M*(m+1) (RPE of finished walks)
    wl = synth.Workload("t", "rmat", 4096, 60_000, 0.0, M, m, 0, 2, "uniform", graph_seed=M)
    rp, ci = synth.make_graph(wl)
    seeds = np.concatenate([np.arange(4096), np.arange(1500)]).astype(np.int32)
    w = oracle.sample_walks(rp, ci, seeds, M, m, 5)
    t_off, t_ids, t_cnt = oracle.build_rpe(w)
    for n in (seeds.size, 600):
        rows = int(t_off[n])
        walks, off, ids, cnt = binding.sample_walks_rpe(ctx, dev(rp), dev(ci), dev(seeds[:n]), M, m, 5)
        assert np.array_equal(walks.cpu().numpy(), w[:n])
        b_off, b_ids, b_cnt = binding.build_rpe(ctx, walks, wl.n_nodes)
        assert ctx.check() == 0
        for o, i, c in ((off, ids, cnt), (b_off, b_ids, b_cnt)):
            assert np.array_equal(o.cpu().numpy(), t_off[:n + 1])
            assert np.array_equal(i.cpu().numpy(), t_ids[:rows])
            assert np.array_equal(host_u16(c).reshape(-1, m + 1), t_cnt[:rows])


@pytest.mark.parametrize("L", [2, 3, 4, 5, 6])
@pytest.mark.parametrize("n_T", [32_766, 32_767, 32_768, 42_000, 50_001, 70_711])
def test_prune_numbers_of_16_bits(ctx, L, n_T):
    # on both sides of the number of vectors whose numbers fit 16 bits; most rows have common vectors and
    # every tile some rare ones, so that rows whose numbers do not fit lie in tiles that went out in 16 bits,
    # in ones that did not, and behind the last whole tile; ranked all with all and by the sort (from 70,711
    # vectors of two counts, 50,001 of three or four and 40,825 of five or six)
    n_rows = 6_000_000 + 77
    g = torch.Generator(device="cuda").manual_seed(n_T + L)
    number = torch.randperm(n_T, device="cuda", generator=g)
    vectors = torch.randint(0, 4, (n_T, L), device="cuda", generator=g)
    vectors[:, 0], vectors[:, -1] = number % 256, number // 256
    pick = (torch.rand(n_rows, device="cuda", generator=g) * 40).long()
    rare = torch.rand(n_rows, device="cuda", generator=g) < 0.02
    pick[rare] = torch.randint(0, n_T, (int(rare.sum()),), device="cuda", generator=g)
    pick[torch.randperm(n_rows, device="cuda", generator=g)[:n_T]] = torch.arange(n_T, device="cuda")
    cnt = vectors[pick].to(torch.int16).contiguous().view(torch.uint16)
    want = torch.unique(vectors, dim=0)
    assert want.shape[0] == n_T
    T = torch.zeros((1 << 17, L), dtype=torch.int16, device="cuda").view(torch.uint16)
    codes = torch.zeros(n_rows + 3, dtype=torch.int32, device="cuda")
    for place in range(4):  # codes that start anywhere; later calls find the set empty again
        code = codes[place:place + n_rows]
        rc, got = binding.prune_rpe_raw(ctx, cnt, 1 << 17, T, code)
        assert rc == binding.OK and got == n_T and ctx.check() == 0
        assert torch.equal(T.view(torch.int16)[:n_T].long(), want)
        assert torch.equal(T.view(torch.int16)[code.long()], cnt.view(torch.int16))


@pytest.mark.parametrize("L", [2, 4, 5])
@pytest.mark.parametrize("n_T", [32_767, 32_768, 40_001])
def test_pruning_has_done_its_work_when_it_returns(ctx, L, n_T):
    # the call waits for its own work, also where the hash set is emptied by a launch of its own (more vectors
    # than 16-bit numbers, fewer than are sorted): nothing of it is still under way on the stream
    number = torch.arange(n_T, device="cuda")
    vectors = torch.zeros((n_T, L), dtype=torch.int64, device="cuda")
    vectors[:, 0], vectors[:, -1] = number % 256, number // 256
    cnt = vectors.to(torch.int16).contiguous().view(torch.uint16)
    T = torch.zeros((1 << 17, L), dtype=torch.int16, device="cuda").view(torch.uint16)
    code = torch.zeros(n_T, dtype=torch.int32, device="cuda")
    busy = 0
    for _ in range(40):
        rc, got = binding.prune_rpe_raw(ctx, cnt, 1 << 17, T, code)
        busy += not ctx.stream.query()
        assert rc == binding.OK and got == n_T
    assert busy == 0 and ctx.check() == 0


def test_one_call_rpe_ids_of_many_distinct_vectors(ctx):
    # every node is visited several times at every step, so hardly two rows are the same
    wl = synth.Workload("t", "rmat", 256, 5000, 0.0, 128, 15, 0, 2, "uniform", graph_seed=3)
    rp, ci = synth.make_graph(wl)
    seeds = np.arange(wl.n_nodes, dtype=np.int32)
    w = oracle.sample_walks(rp, ci, seeds, wl.M, wl.m, 6)
    t_off, t_ids, t_cnt = oracle.build_rpe(w)
    want_T, want_code = oracle.prune_rpe(t_cnt)
    assert want_T.shape[0] > 25_000
    _, off, ids, cnt, code, T = binding.sample_walks_rpe_ids(ctx, dev(rp), dev(ci), dev(seeds), wl.M,
                                                             wl.m, 6, cap_T=1 << 17)
    assert ctx.check() == 0
    assert np.array_equal(ids.cpu().numpy(), t_ids) and np.array_equal(off.cpu().numpy(), t_off)
    assert np.array_equal(host_u16(T).reshape(want_T.shape), want_T)
    assert np.array_equal(code.cpu().numpy(), want_code)


def test_query_rpe_ids_problems_are_flagged(ctx):
    wl = synth.Workload("t", "rmat", 256, 900, 0.0, 20, 3, 0, 2, "uniform", graph_seed=3)
    rp, ci = synth.make_graph(wl)
    seeds = np.arange(32, dtype=np.int32)
    walks, off, ids, cnt = binding.sample_walks_rpe(ctx, dev(rp), dev(ci), dev(seeds), wl.M, wl.m, 0)
    q = np.array([[1, 2], [5, 32], [3, 4]], dtype=np.int32)          # 32 is not a block
    got = binding.query_rpe_ids(ctx, walks, off, ids, dev(q), max_set=61).cpu().numpy()
    assert ctx.check() == binding.DEV_BAD_QUERY
    assert (got[1] == -1).all()
    want = oracle.query_rpe_ids(walks.cpu().numpy(), off.cpu().numpy(), ids.cpu().numpy(),
                                q[[0, 2]])
    assert np.array_equal(got[[0, 2]].astype(np.int64), want)
    sizes = np.diff(off.cpu().numpy())
    big = int(np.argmax(sizes))
    got = binding.query_rpe_ids(ctx, walks, off, ids, dev(np.array([[big, 0]], np.int32)),
                                max_set=int(sizes[big]) - 1)
    assert ctx.check() == binding.DEV_SET_TOO_LARGE and bool((got == -1).all())


@pytest.mark.parametrize("k,M,m", [(2, 13, 4), (2, 100, 4), (2, 204, 4), (3, 60, 2), (3, 400, 4)])
def test_query_rpe_ids_of_crowded_and_even_id_lists(ctx, k, M, m):
    # hand-made walks whose blocks' ids lie evenly in their range, crowd together at one end with
    # one id far away, follow one another, are all the same, or lie far above everybody else's:
    # the look-up's directory and its bisection, walk blocks of one and several rounds
    rng = np.random.default_rng(M + k)
    n_nodes = 1 << 27
    sets = [rng.choice(n_nodes, 300, replace=False), np.r_[np.arange(280), n_nodes - 1],
            np.arange(5000, 5300), np.array([77]), np.arange(n_nodes - 200, n_nodes),
            np.r_[np.arange(0, 3000, 30), np.arange(100000, 100009), 70000000], np.array([0, n_nodes - 1])]
    blocks = [s[rng.integers(0, s.size, size=(M, m + 1))] for s in sets]
    blocks += [np.concatenate([b[: M // 2], c[M // 2:]]) for b, c in zip(blocks, blocks[1:])]
    walks = np.stack(blocks).astype(np.int32)
    off, ids, cnt = oracle.build_rpe(walks)
    queries = rng.integers(0, len(blocks), size=(200, k)).astype(np.int32)
    max_set = int(np.diff(off).max())
    code = rng.integers(0, 1 << 30, size=ids.size).astype(np.int32)
    want = oracle.query_rpe_ids(walks, off, ids, queries)
    got = binding.query_rpe_ids(ctx, dev(walks), dev(off), dev(ids), dev(queries), max_set)
    assert ctx.check() == 0
    assert np.array_equal(got.cpu().numpy().astype(np.int64), want)
    got = binding.query_rpe_ids(ctx, dev(walks), dev(off), dev(ids), dev(queries), max_set, code=dev(code))
    assert ctx.check() == 0
    assert np.array_equal(got.cpu().numpy(), np.where(want < 0, -1, code[want]))


def test_join_problems_are_flagged(ctx):
    wl = synth.Workload("t", "rmat", 256, 900, 0.0, 20, 3, 0, 2, "uniform", graph_seed=3)
    rp, ci = synth.make_graph(wl)
    seeds = np.arange(32, dtype=np.int32)
    out = gpu_pipeline(ctx, rp, ci, seeds, wl.M, wl.m, 0)
    off, ids, cnt = out["rpe"]
    table = oracle.build_rpe(out["walks"].cpu().numpy())
    good = np.array([[1, 2], [3, 4]], dtype=np.int32)
    want = oracle.join_queries(*table, good)
    # a query entry outside the table: that query yields no rows, the others are intact
    q = np.array([[1, 2], [5, 32], [-1, 0], [3, 4]], dtype=np.int32)
    joff, jids, jcnt = binding.join_queries(ctx, off, ids, cnt, dev(q), max_set=61)
    assert ctx.check() == binding.DEV_BAD_QUERY
    joff_h = joff.cpu().numpy()
    assert joff_h[2] == joff_h[1] and joff_h[3] == joff_h[2]
    assert np.array_equal(jids.cpu().numpy(), want[1])
    assert np.array_equal(host_u16(jcnt), want[2])
    # max_set smaller than a queried block
    sizes = np.diff(table[0])
    big = int(np.argmax(sizes))
    assert sizes[big] >= 2
    joff, jids, jcnt = binding.join_queries(ctx, off, ids, cnt,
                                            dev(np.array([[big, big]], np.int32)),
                                            max_set=int(sizes[big]) - 1)
    assert ctx.check() == binding.DEV_SET_TOO_LARGE
    assert jids.numel() == 0
    # capacity
    joff = torch.empty(3, dtype=torch.int64, device="cuda")
    total = int(want[0][-1])
    jids = torch.full((total,), -7, dtype=torch.int32, device="cuda")
    jcnt = torch.zeros((total, 2, 4), dtype=torch.int16, device="cuda").view(torch.uint16)
    cap = int(want[0][1])                                    # room for the first query only
    rc, rows = binding.join_queries_raw(ctx, off, ids, cnt, dev(good), 61, cap, joff, jids, jcnt)
    assert rc == binding.E_CAPACITY and rows == total
    assert ctx.check() == binding.DEV_CAPACITY
    assert np.array_equal(jids.cpu().numpy()[:cap], want[1][:cap])
    assert (jids.cpu().numpy()[cap:] == -7).all()


# --------------------------------------------------------------------------- #
# the two phases as calls of their own: size, allocate, fill
# --------------------------------------------------------------------------- #
@pytest.mark.parametrize("M,m,k", [(50, 4, 2), (200, 3, 3), (33, 2, 2), (20, 7, 3)])
def test_count_then_fill_calls_against_the_oracle(ctx, M, m, k):
    wl = synth.Workload("t", "rmat", 2048, 12000, 0.0, M, m, 0, k, "uniform", graph_seed=21)
    rp, ci = synth.make_graph(wl)
    rng = np.random.default_rng(M + m)
    seeds = rng.integers(0, wl.n_nodes, size=777).astype(np.int32)
    queries = rng.integers(0, seeds.size, size=(1501, k)).astype(np.int32)
    L = m + 1
    w = oracle.sample_walks(rp, ci, seeds, M, m, 9)
    table = oracle.build_rpe(w)
    joined = oracle.join_queries(*table, queries)

    walks = binding.sample_walks(ctx, dev(rp), dev(ci), dev(seeds), M, m, 9)
    off = torch.empty(seeds.size + 1, dtype=torch.int64, device="cuda")
    rc, R = binding.build_rpe_count(ctx, walks, wl.n_nodes, off)
    assert rc == binding.OK and R == table[1].size
    assert np.array_equal(off.cpu().numpy(), table[0])
    ids = torch.empty(R, dtype=torch.int32, device="cuda")
    cnt = torch.empty((R, L), dtype=torch.uint16, device="cuda")
    kept = off.clone()
    assert binding.build_rpe_fill(ctx, walks, wl.n_nodes, off, R, ids, cnt) == binding.OK
    assert ctx.check() == 0
    assert torch.equal(off, kept), "the filling call changed the offsets it was given"
    assert_table_equal((off, ids, cnt), table, "rpe by count + fill")

    d_q = dev(queries)
    joff = torch.empty(queries.shape[0] + 1, dtype=torch.int64, device="cuda")
    rc, J = binding.join_count(ctx, off, ids, d_q, 1 + M * m, joff)
    assert rc == binding.OK and J == joined[1].size
    jids = torch.empty(J, dtype=torch.int32, device="cuda")
    jcnt = torch.empty((J, k, L), dtype=torch.uint16, device="cuda")
    kept = joff.clone()
    assert binding.join_fill(ctx, off, ids, cnt, d_q, 1 + M * m, joff, J, jids, jcnt) == binding.OK
    assert ctx.check() == 0
    assert torch.equal(joff, kept)
    assert_table_equal((joff, jids, jcnt), joined, "join by count + fill")
    # offsets kept from an earlier call fill again without any counting
    jids.fill_(-7)
    assert binding.join_fill(ctx, off, ids, cnt, d_q, 1 + M * m, joff, J, jids, jcnt) == binding.OK
    assert ctx.check() == 0
    assert np.array_equal(jids.cpu().numpy(), joined[1])


def test_fill_calls_with_offsets_of_something_else_are_flagged(ctx):
    wl = synth.Workload("t", "rmat", 256, 900, 0.0, 20, 3, 0, 2, "uniform", graph_seed=3)
    rp, ci = synth.make_graph(wl)
    seeds = np.arange(40, dtype=np.int32)
    walks, off, ids, cnt = binding.sample_walks_rpe(ctx, dev(rp), dev(ci), dev(seeds), wl.M, wl.m, 0)
    table = oracle.build_rpe(walks.cpu().numpy())
    q = np.array([[1, 2], [3, 4], [5, 6], [7, 8]], dtype=np.int32)
    want = oracle.join_queries(*table, q)
    joff = torch.from_numpy(want[0].copy()).cuda()
    joff[2:] += 2                                      # query 1 is given two rows too many
    total = int(joff[-1])
    jids = torch.full((total,), -7, dtype=torch.int32, device="cuda")
    jcnt = torch.zeros((total, 2, 4), dtype=torch.int16, device="cuda").view(torch.uint16)
    assert binding.join_fill(ctx, off, ids, cnt, dev(q), 61, joff, total, jids, jcnt) == binding.OK
    assert ctx.check() == binding.DEV_BAD_SIZES
    got = jids.cpu().numpy()
    lo, hi = int(want[0][1]), int(want[0][2]) + 2
    assert (got[lo:hi] == -7).all()                    # the mismatched query wrote nothing
    assert np.array_equal(got[:lo], want[1][:lo])      # the others are where the offsets put them
    assert np.array_equal(got[hi:], want[1][int(want[0][2]):])
    # the same for the table's rows
    roff = torch.from_numpy(table[0].copy()).cuda()
    roff[6:] += 1
    total = int(roff[-1])
    rids = torch.full((total,), -7, dtype=torch.int32, device="cuda")
    rcnt = torch.zeros((total, 4), dtype=torch.int16, device="cuda").view(torch.uint16)
    assert binding.build_rpe_fill(ctx, walks, wl.n_nodes, roff, total, rids, rcnt) == binding.OK
    assert ctx.check() == binding.DEV_BAD_SIZES
    got = rids.cpu().numpy()
    lo, hi = int(table[0][5]), int(table[0][6]) + 1
    assert (got[lo:hi] == -7).all()
    assert np.array_equal(got[:lo], table[1][:lo]) and np.array_equal(got[hi:], table[1][int(table[0][6]):])


@pytest.mark.parametrize("n_seeds", [50, 5000])
def test_bad_seeds_give_the_same_table_on_both_paths(ctx, n_seeds):
    # a seed that is not a node gets walks of -1 and no rows, whether the table is built by the
    # fused kernel or by surel_build_rpe over those walks
    wl = synth.Workload("t", "rmat", 256, 900, 0.0, 20, 3, 0, 2, "uniform", graph_seed=3)
    rp, ci = synth.make_graph(wl)
    seeds = np.arange(n_seeds, dtype=np.int32) % wl.n_nodes
    seeds[[0, 17, n_seeds - 1]] = [-1, 256, 1 << 30]
    good = np.ones(n_seeds, dtype=bool)
    good[[0, 17, n_seeds - 1]] = False
    d_rp, d_ci, d_seeds = dev(rp), dev(ci), dev(seeds)
    f_walks, f_off, f_ids, f_cnt = binding.sample_walks_rpe(ctx, d_rp, d_ci, d_seeds, wl.M, wl.m, 2)
    assert ctx.check() == binding.DEV_BAD_SEED
    for sizes in (None, torch.empty(n_seeds, dtype=torch.int32, device="cuda")):
        walks = binding.sample_walks(ctx, d_rp, d_ci, d_seeds, wl.M, wl.m, 2, set_sizes=sizes)
        assert ctx.check() == binding.DEV_BAD_SEED
        off, ids, cnt = binding.build_rpe(ctx, walks, wl.n_nodes, set_sizes=sizes)
        assert ctx.check() == binding.DEV_BAD_WALK          # the -1 entries are left out, and said so
        assert torch.equal(walks, f_walks) and torch.equal(off, f_off) and torch.equal(ids, f_ids)
        assert torch.equal(cnt.view(torch.int16), f_cnt.view(torch.int16))
    w = oracle.sample_walks(rp, ci, seeds[good], wl.M, wl.m, 2)
    t_off, t_ids, t_cnt = oracle.build_rpe(w)
    sizes_h = np.zeros(n_seeds, dtype=np.int64)
    sizes_h[good] = np.diff(t_off)
    assert np.array_equal(f_off.cpu().numpy(), np.concatenate([[0], np.cumsum(sizes_h)]))
    assert np.array_equal(f_ids.cpu().numpy(), t_ids) and np.array_equal(host_u16(f_cnt), t_cnt)


@pytest.mark.parametrize("k", [2, 3])
def test_join_query_counts_around_workgroup_and_scan_tile_sizes(ctx, k):
    # 4 waves a workgroup, 2048 counts per tile of the offset scan: query counts on and around
    # those sizes against the oracle
    wl = synth.Workload("t", "rmat", 2048, 12000, 0.0, 50, 4, 0, k, "uniform", graph_seed=5)
    rp, ci = synth.make_graph(wl)
    seeds = np.arange(wl.n_nodes, dtype=np.int32)
    walks, off, ids, cnt = binding.sample_walks_rpe(ctx, dev(rp), dev(ci), dev(seeds), wl.M, wl.m, 4)
    table = oracle.build_rpe(walks.cpu().numpy())
    rng = np.random.default_rng(k)
    all_q = rng.integers(0, wl.n_nodes, size=(20000, k)).astype(np.int32)
    for n in (1, 2, 7, 8, 9, 15, 16, 17, 31, 33, 64, 2047, 2048, 2049, 4104, 16391, 20000):
        want = oracle.join_queries(*table, all_q[:n])
        got = binding.join_queries(ctx, off, ids, cnt, dev(all_q[:n]), max_set=201,
                                   cap_rows=int(want[0][-1]) + 5)
        assert ctx.check() == 0
        assert_table_equal(got, want, f"join of {n} queries")


def hand_made_table(blocks, L, rng):
    """An RPE table whose blocks hold the given ascending id lists and random counts."""
    off = np.zeros(len(blocks) + 1, dtype=np.int64)
    off[1:] = np.cumsum([len(b) for b in blocks])
    ids = np.concatenate([np.asarray(b, dtype=np.int32) for b in blocks]) if off[-1] else \
        np.zeros(0, dtype=np.int32)
    cnt = rng.integers(0, 65536, size=(int(off[-1]), L)).astype(np.uint16)
    return off, ids, cnt


@pytest.mark.parametrize("max_set", [1, 31, 32, 33, 64, 96, 2048])
@pytest.mark.parametrize("L", [2, 4, 5, 7])
def test_join_of_hand_made_tables_around_64_row_boundaries(ctx, max_set, L):
    # pairs whose unions end exactly at, one before and one after a multiple of 64 rows (the
    # union's bit masks are 64-bit words; a round of the filling loop is 64 rows), from lists
    # that are disjoint, equal, interleaved, nested, empty, and full sets of max_set nodes
    rng = np.random.default_rng(1000 * max_set + L)
    n = max_set
    even, odd = np.arange(0, 2 * n, 2), np.arange(1, 2 * n, 2)
    low, high = np.arange(n), np.arange(n, 2 * n)
    blocks = [even, odd, low, high, low[: n // 2], low[n // 2:], np.zeros(0, dtype=np.int64),
              low[:1], high[-1:], even[: max(n - 1, 0)], np.sort(rng.choice(4 * n, n, replace=False)),
              np.sort(rng.choice(4 * n, n, replace=False))]
    table = hand_made_table(blocks, L, rng)
    nb = len(blocks)
    queries = np.array([(a, b) for a in range(nb) for b in range(nb)], dtype=np.int32)
    want = oracle.join_queries(*table, queries)
    sizes = np.diff(want[0])
    assert sizes.max() == 2 * n and (sizes == 0).any()
    d_table = (dev(table[0]), dev(table[1]), dev(table[2].view(np.int16)).view(torch.uint16))
    got = binding.join_queries(ctx, *d_table, dev(queries), max_set=max_set)
    assert ctx.check() == 0
    assert_table_equal(got, want, f"hand-made join, max_set {max_set}, L {L}")
    if max_set > 96:
        return
    # and as triples: (a, b, b) and (a, a, b) have the union of (a, b) with a list repeated
    tri = np.concatenate([queries[:, [0, 1, 1]], queries[:, [0, 0, 1]]])[:: 3]
    want3 = oracle.join_queries(*table, tri)
    got3 = binding.join_queries(ctx, *d_table, dev(tri), max_set=max_set)
    assert ctx.check() == 0
    assert_table_equal(got3, want3, f"hand-made join of triples, max_set {max_set}, L {L}")


@pytest.mark.parametrize("k", [2, 3])
@pytest.mark.parametrize("L", [2, 3, 6, 7, 8, 9, 10, 13, 15, 16])
def test_join_vector_lengths_in_one_and_in_two_launches(ctx, L, k):
    # every kind of row (whole words, rows that straddle words) of short and long vectors, from
    # unions that end around multiples of 64 rows; few queries take one launch with several waves
    # to a query, many take two with one wave each: same rows
    rng = np.random.default_rng(10 * L + k)
    n = 96
    blocks = [np.sort(rng.choice(3 * n, size, replace=False)) for size in (96, 95, 64, 63, 33, 1, 0, 80)]
    table = hand_made_table(blocks, L, rng)
    d_table = (dev(table[0]), dev(table[1]), dev(table[2].view(np.int16)).view(torch.uint16))
    few = rng.integers(0, len(blocks), size=(333, k)).astype(np.int32)
    many = np.concatenate([few] * 13)
    assert few.shape[0] < 4096 < many.shape[0]
    for queries in (few, many):
        want = oracle.join_queries(*table, queries)
        got = binding.join_queries(ctx, *d_table, dev(queries), max_set=n)
        assert ctx.check() == 0
        assert_table_equal(got, want, f"join of {queries.shape[0]} {k}-tuples, L {L}")


@pytest.mark.parametrize("k", [2, 3])
@pytest.mark.parametrize("L", [2, 4, 5, 10])
def test_join_fill_at_every_place_of_a_line(ctx, L, k):
    # blocks of sizes that put queries at every place inside 32 rows of the output, and outputs that
    # start anywhere in a line: small ones, which are written through the caches
    rng = np.random.default_rng(100 * L + k)
    sizes = [0, 1, 2, 15, 16, 31, 32, 33, 47, 63, 64, 65, 95, 96]
    blocks = [np.sort(rng.choice(300, size, replace=False)) for size in sizes]
    table = hand_made_table(blocks, L, rng)
    d_table = (dev(table[0]), dev(table[1]), dev(table[2].view(np.int16)).view(torch.uint16))
    queries = rng.integers(0, len(blocks), size=(2500, k)).astype(np.int32)
    want = oracle.join_queries(*table, queries)
    J, d_q, d_off = want[1].size, dev(queries), dev(want[0])
    assert set(np.unique(want[0] % 32)) == set(range(32))
    for skip in (0, 1, 5, 32) if k * L % 2 == 0 else (0, 2, 6, 32):  # outputs are aligned words
        ids = torch.full((J + 64,), -7, dtype=torch.int32, device="cuda")
        cnt = torch.full((J + 64, k, L), 9, dtype=torch.int16, device="cuda").view(torch.uint16)
        part = slice(skip, skip + J)
        assert binding.join_fill(ctx, *d_table, d_q, 96, d_off, J, ids[part], cnt[part]) == binding.OK
        assert ctx.check() == 0
        assert_table_equal((d_off, ids[part], cnt[part]), want, f"rows from place {skip} on")
        for rest in (slice(0, skip), slice(skip + J, None)):
            assert (ids[rest] == -7).all() and (cnt.view(torch.int16)[rest] == 9).all()


@pytest.mark.parametrize("k", [2, 3])
@pytest.mark.parametrize("L", range(2, 17))
def test_join_fill_past_the_caches_at_every_place_of_a_line(ctx, L, k):
    # an output of so many bytes is written past the caches, a query's rows from their place inside 32
    # rows of the lines on: queries at every such place, for every length of vector, in outputs that
    # start anywhere in a line, ids and vectors at the same row and at different ones
    lines = open(os.path.join(os.path.dirname(binding.LIB_PATH), "csrc", "lines.h")).read()
    a, shift = re.search(r"kPastBytes = (\d+) << (\d+);", lines).groups()
    past = int(a) << int(shift)
    rng = np.random.default_rng(100 * L + k)
    sizes = [0, 1, 2, 15, 16, 31, 32, 33, 47, 63, 64, 65, 95, 96, 400]
    blocks = [np.sort(rng.choice(900, size, replace=False)) for size in sizes]
    table = hand_made_table(blocks, L, rng)
    d_table = (dev(table[0]), dev(table[1]), dev(table[2].view(np.int16)).view(torch.uint16))
    queries = rng.integers(0, len(blocks), size=(2500, k)).astype(np.int32)
    want = oracle.join_queries(*table, queries)
    J, row_bytes = want[1].size, 4 + 2 * k * L
    times = past // (J * row_bytes) + 1  # the list of queries over and over
    assert times * J * row_bytes > past
    d_q = dev(queries).repeat(times, 1)
    d_off = dev(want[0])
    starts = (torch.arange(times, device="cuda") * J).view(-1, 1) + d_off[:-1]
    d_off = torch.cat([starts.flatten(), torch.tensor([times * J], device="cuda")])
    assert (d_off[:-1] % 32).unique().numel() == 32
    w_ids, w_cnt = dev(want[1]), dev(want[2].view(np.int16)).view(J, k, L)
    rows = times * J
    ids = torch.empty(rows + 64, dtype=torch.int32, device="cuda")
    cnt = torch.empty((rows + 64, k, L), dtype=torch.int16, device="cuda")
    even = k * L % 2 == 0  # vectors of an output start at aligned words
    for at_ids, at_cnt in ((0, 0), (1, 1) if even else (2, 2), (38, 38), (0, 6), (5, 0)):
        ids.fill_(-7), cnt.fill_(9)
        in_ids, in_cnt = ids[at_ids:at_ids + rows], cnt[at_cnt:at_cnt + rows]
        assert binding.join_fill(ctx, *d_table, d_q, 400, d_off, rows, in_ids,
                                 in_cnt.view(torch.uint16)) == binding.OK
        assert ctx.check() == 0
        assert bool((in_ids.view(times, J) == w_ids).all()), f"ids from place {at_ids} on"
        assert bool((in_cnt.view(times, J, k, L) == w_cnt).all()), f"vectors from place {at_cnt} on"
        assert (ids[:at_ids] == -7).all() and (ids[at_ids + rows:] == -7).all()
        assert (cnt[:at_cnt] == 9).all() and (cnt[at_cnt + rows:] == 9).all()


@pytest.mark.parametrize("k", [2, 3])
@pytest.mark.parametrize("stride", [1, 3, 1 << 13, 1 << 17])
def test_join_counts_of_lists_whose_ids_share_bits(ctx, stride, k):
    # the counting launch looks ids up in a bit map of hashed ids first: ids next to each other, in
    # even steps, and 2^24 apart (which share a bit), in lists around the 64 ids of a register, the
    # 512 ids that the registers hold, and the largest
    rng = np.random.default_rng(stride + k)
    limit = (1 << 28) // stride - 1
    far = (1 << 24) // stride
    blocks = []
    for size in (0, 1, 63, 64, 65, 200, 511, 512, 513, 1024, 2047, 2048):
        span = min(4096, limit)
        near = rng.choice(span, min(size, span), replace=False)
        blocks.append(np.sort(near) * stride)
        if far and size <= 512:  # every other id 2^24 further on
            near = near + np.where(np.arange(near.size) % 2 == 1, far, 0)
            blocks.append(np.unique(near) * stride)
    table = hand_made_table(blocks, 2, rng)
    queries = rng.integers(0, len(blocks), size=(4500, k)).astype(np.int32)
    want = oracle.join_queries(*table, queries)
    off = torch.empty(queries.shape[0] + 1, dtype=torch.int64, device="cuda")
    rc, J = binding.join_count(ctx, dev(table[0]), dev(table[1]), dev(queries), 2048, off)
    assert rc == binding.OK and ctx.check() == 0 and J == want[1].size
    assert np.array_equal(off.cpu().numpy(), want[0])
    # lists of so many queries that a wavefront has several of them, up to its eight and with a rest,
    # the next one's ids on their way while one is counted: the sizes are those of the unions
    of = {tuple(q): n for q, n in zip(queries.tolist(), np.diff(want[0]).tolist())}
    for q in itertools.product(range(len(blocks)), repeat=k):
        if q not in of:
            of[q] = np.unique(np.concatenate([blocks[b] for b in q])).size
    per_cu = 16 * torch.cuda.get_device_properties(0).multi_processor_count
    for n in (2 * per_cu + 1, 5 * per_cu + 3, 8 * per_cu, 9 * per_cu + 5):
        queries = rng.integers(0, len(blocks), size=(n, k)).astype(np.int32)
        off = torch.empty(n + 1, dtype=torch.int64, device="cuda")
        rc, J = binding.join_count(ctx, dev(table[0]), dev(table[1]), dev(queries), 2048, off)
        sizes = np.array([of[tuple(q)] for q in queries.tolist()])
        assert rc == binding.OK and ctx.check() == 0 and J == sizes.sum()
        assert np.array_equal(np.diff(off.cpu().numpy()), sizes)


@pytest.mark.parametrize("k", [2, 3])
def test_join_in_one_launch_of_the_largest_blocks_and_with_bounded_waits(ctx, k):
    # full blocks of 2048 rows; with no wait allowed at all a workgroup unites the lists that it
    # would have waited for itself: the offsets are right all the same
    rng = np.random.default_rng(k)
    blocks = [np.sort(rng.choice(9000, 2048, replace=False)) for _ in range(4)]
    table = hand_made_table(blocks, 5, rng)
    d_table = (dev(table[0]), dev(table[1]), dev(table[2].view(np.int16)).view(torch.uint16))
    queries = rng.integers(0, 4, size=(300, k)).astype(np.int32)
    want = oracle.join_queries(*table, queries)
    joff = torch.empty(queries.shape[0] + 1, dtype=torch.int64, device="cuda")
    for spins in (1 << 22, 0, 1 << 22):
        ctx.set_spin_limit(spins)
        try:
            rc, rows = binding.join_queries_raw(ctx, *d_table, dev(queries), 2048, 0, joff, None, None)
        finally:
            ctx.set_spin_limit(1 << 22)
        assert rc == binding.OK and rows == want[0][-1] and ctx.check() == 0
        assert np.array_equal(joff.cpu().numpy(), want[0])
    got = binding.join_queries(ctx, *d_table, dev(queries), max_set=2048)
    assert ctx.check() == 0
    assert_table_equal(got, want, "join of full blocks")


@pytest.mark.parametrize("spins", [0, 1, 2, 5])
def test_launches_that_add_up_each_others_counts_depend_on_no_wait(ctx, spins):
    # walks + RPE of few seeds, joins of few queries, offset scans and the incidence sort with
    # (nearly) no poll allowed: whoever finds a count missing works it out itself, so the call is
    # complete and says OK
    wl = synth.Workload("t", "rmat", 16384, 100000, 0.0, 50, 4, 0, 2, "uniform", graph_seed=9)
    rp, ci = synth.make_graph(wl)
    d_rp, d_ci = dev(rp), dev(ci)
    M, m, L = wl.M, wl.m, wl.m + 1
    rng = np.random.default_rng(spins)
    all_seeds = np.arange(wl.n_nodes, dtype=np.int32)
    w = oracle.sample_walks(rp, ci, all_seeds, M, m, 1)
    t_off, t_ids, t_cnt = oracle.build_rpe(w)
    ctx.set_spin_limit(spins)
    try:
        for S in (1, 2, 63, 257, 1000, 4095, 4096):
            cap = int(t_off[S])
            walks = torch.empty((S, M, L), dtype=torch.int32, device="cuda")
            off = torch.full((S + 1,), -7, dtype=torch.int64, device="cuda")
            ids = torch.full((cap,), -7, dtype=torch.int32, device="cuda")
            cnt = torch.zeros((cap, L), dtype=torch.int16, device="cuda").view(torch.uint16)
            rc, rows = binding.sample_walks_rpe_raw(ctx, d_rp, d_ci, dev(all_seeds[:S]), M, m, 1,
                                                    walks, cap, off, ids, cnt)
            assert rc == binding.OK and rows == cap and ctx.check() == 0, f"{S} seeds"
            assert np.array_equal(walks.cpu().numpy(), w[:S])
            assert_table_equal((off, ids, cnt), (t_off[:S + 1], t_ids[:cap], t_cnt[:cap]), f"{S} seeds")
        # the two calls, with the scan of 16,384 counts in two workgroups
        off, ids, cnt = binding.build_rpe(ctx, dev(w), wl.n_nodes)
        assert ctx.check() == 0
        assert_table_equal((off, ids, cnt), (t_off, t_ids, t_cnt), "build_rpe")
        for k in (2, 3):
            for n_q in (1, 33, 300, 2049, 4096):
                queries = rng.integers(0, wl.n_nodes, size=(n_q, k)).astype(np.int32)
                want = oracle.join_queries(t_off, t_ids, t_cnt, queries)
                got = binding.join_queries(ctx, off, ids, cnt, dev(queries), max_set=1 + M * m)
                assert ctx.check() == 0, f"{n_q} {k}-tuples"
                assert_table_equal(got, want, f"join of {n_q} {k}-tuples")
        # 30,000 queries: 15 tiles a pass of the sort; 300,000: tiles of the larger kind
        for n_q in (30_000, 300_000):
            queries = rng.integers(0, wl.n_nodes, size=(n_q, 2)).astype(np.int32)
            inc_off, inc_q = binding.query_incidence(ctx, dev(queries), wl.n_nodes)
            assert ctx.check() == 0
            flat = queries.reshape(-1)
            order = np.argsort(flat, kind="stable")
            assert np.array_equal(inc_q.cpu().numpy(), order // 2)
            assert np.array_equal(inc_off.cpu().numpy(),
                                  np.searchsorted(flat[order], np.arange(wl.n_nodes + 1)))
    finally:
        ctx.set_spin_limit(1 << 22)


@pytest.mark.parametrize("M,m", [(1, 1), (65, 3), (128, 15), (200, 9)])
def test_helpers_count_what_the_owners_count(ctx, M, m):
    # no poll allowed: walk blocks of every size, seeds that are no nodes, blocks that are empty,
    # queries that name none, in the places that helpers work out
    wl = synth.Workload("t", "rmat", 512, 3000, 0.0, M, m, 0, 2, "uniform", graph_seed=4)
    rp, ci = synth.make_graph(wl)
    rng = np.random.default_rng(M)
    seeds = rng.integers(0, wl.n_nodes, size=1000).astype(np.int32)
    seeds[::7] = [-1, wl.n_nodes, 1 << 30][M % 3]
    queries = rng.integers(0, seeds.size, size=(700, 3)).astype(np.int32)
    queries[::5, 1] = queries[::5, 0]
    queries[3::11, 2] = seeds.size
    d_rp, d_ci, d_seeds, d_q = dev(rp), dev(ci), dev(seeds), dev(queries)
    got = []
    for spins in (1 << 22, 0):
        ctx.set_spin_limit(spins)
        try:
            walks, off, ids, cnt = binding.sample_walks_rpe(ctx, d_rp, d_ci, d_seeds, M, m, 2)
            assert ctx.check() == binding.DEV_BAD_SEED
            joff, jids, jcnt = binding.join_queries(ctx, off, ids, cnt, d_q, max_set=1 + M * m)
            assert ctx.check() == binding.DEV_BAD_QUERY
        finally:
            ctx.set_spin_limit(1 << 22)
        got.append([walks, off, ids, cnt.view(torch.int16), joff, jids, jcnt.view(torch.int16)])
    for a, b in zip(*got):
        assert torch.equal(a, b)
    w = oracle.sample_walks(rp, ci, seeds[seeds != seeds[0]], M, m, 2)
    assert int(got[0][1][-1]) == oracle.build_rpe(w)[1].size


def test_small_calls_of_three_contexts_at_a_time():
    # three contexts on streams of their own, each with launches that would fill the device alone,
    # enqueued in turn without waiting: every call's rows are complete
    wl = synth.Workload("t", "rmat", 4096, 30000, 0.0, 50, 4, 0, 2, "uniform", graph_seed=9)
    rp, ci = synth.make_graph(wl)
    M, m, L, S, rounds = wl.M, wl.m, wl.m + 1, wl.n_nodes, 8
    rng = np.random.default_rng(2)
    queries = rng.integers(0, S, size=(4096, 2)).astype(np.int32)
    jobs = []
    for i in range(3):
        w = oracle.sample_walks(rp, ci, np.arange(S, dtype=np.int32), M, m, i)
        table = oracle.build_rpe(w)
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            c = binding.Context(stream=stream)
            cap = table[1].size
            joined = oracle.join_queries(*table, queries)
            J = joined[1].size
            outs = [(torch.empty((S, M, L), dtype=torch.int32, device="cuda"),
                     torch.empty(S + 1, dtype=torch.int64, device="cuda"),
                     torch.full((cap,), -7, dtype=torch.int32, device="cuda"),
                     torch.empty((cap, L), dtype=torch.uint16, device="cuda"),
                     torch.empty(4097, dtype=torch.int64, device="cuda"),
                     torch.full((J,), -7, dtype=torch.int32, device="cuda"),
                     torch.empty((J, 2, L), dtype=torch.uint16, device="cuda")) for _ in range(rounds)]
            jobs.append((i, c, stream, dev(rp), dev(ci), torch.arange(S, dtype=torch.int32, device="cuda"),
                         dev(queries), outs, table, joined))
    torch.cuda.synchronize()
    for r in range(rounds):
        for i, c, stream, d_rp, d_ci, d_seeds, d_q, outs, table, joined in jobs:
            walks, off, ids, cnt, joff, jids, jcnt = outs[r]
            rc, _ = binding.sample_walks_rpe_raw(c, d_rp, d_ci, d_seeds, M, m, i, walks, ids.numel(), off,
                                                 ids, cnt, want_rows=False)
            assert rc == binding.OK
            rc, _ = binding.join_queries_raw(c, off, ids, cnt, d_q, 1 + M * m, jids.numel(), joff, jids,
                                             jcnt, want_rows=False)
            assert rc == binding.OK
    for i, c, stream, _, _, _, _, outs, table, joined in jobs:
        assert c.check() == 0
        for walks, off, ids, cnt, joff, jids, jcnt in outs:
            assert_table_equal((off, ids, cnt), table, f"context {i}")
            assert_table_equal((joff, jids, jcnt), joined, f"join of context {i}")
        c.close()


def test_largest_node_ids(ctx):
    # a graph with the most nodes the library takes (2^28 - 1): the largest ids make sort keys
    # (id << 4 | position) that use all 32 bits and must still sort in front of the padding
    n = binding.MAX_NODES
    top = [n - 1, n - 2, n - 3, n - 4]
    edges = [(a, b) for i, a in enumerate(top) for b in top[i + 1:]]
    edges += [(0, n - 1), (12345, n - 2), (n - 5, 7), (7, 12345)]
    rp, ci = synth.csr_from_edge_list(n, edges)
    seeds = np.array([n - 1, 0, n - 2, 12345, n - 5, 7, n - 3, 5, n - 1], dtype=np.int32)  # 5: isolated
    queries = np.array([[0, 2], [1, 6], [8, 0], [7, 7], [3, 4], [5, 2]], dtype=np.int32)
    out = full_compare(ctx, rp, ci, seeds, 60, 4, 3, queries)
    assert int(out["walks"].max()) == n - 1


def hub_and_ring(n_leaves):
    """Node 0 joined to every one of n_leaves leaves, the leaves joined in a chain."""
    leaf = np.arange(1, n_leaves + 1, dtype=np.int64)
    deg = np.full(n_leaves + 1, 3, dtype=np.int64)
    deg[0], deg[1], deg[n_leaves] = n_leaves, 2, 2
    rp = np.zeros(n_leaves + 2, dtype=np.int64)
    np.cumsum(deg, out=rp[1:])
    ci = np.empty(int(rp[-1]), dtype=np.int32)
    ci[:n_leaves] = leaf
    ci[rp[1:-1]] = 0                                       # every leaf's row: hub, left, right
    ci[rp[2:-1] + 1] = leaf[1:] - 1
    ci[rp[1:-2] + 2 - (leaf[:-1] == 1)] = leaf[:-1] + 1
    return rp.astype(np.int32), ci


def test_packed_edge_records_and_a_degree_beyond_their_field(ctx):
    # the walks read 8-byte neighbour records; the hub's degree (1.2 M) does not fit the 20 bits
    # the record leaves for it and is taken from the CSR
    n_leaves = 1_200_000
    rp, ci = hub_and_ring(n_leaves)
    assert ci.size >= 1 << 22 and np.all(np.diff(rp) > 0)
    rng = np.random.default_rng(5)
    seeds = rng.integers(0, n_leaves + 1, size=50_000, dtype=np.int32)
    seeds[:3] = [0, 1, n_leaves]
    M, m = 200, 3
    assert seeds.size * M * (m - 1) >= 4 * ci.size         # enough steps to make the records
    w = oracle.sample_walks(rp, ci, seeds, M, m, 11)
    assert (w[:, :, 1:] == 0).mean() > 0.2                 # walks do pass through the hub
    table = oracle.build_rpe(w)
    d_rp, d_ci, d_seeds = dev(rp), dev(ci), dev(seeds)
    walks = binding.sample_walks(ctx, d_rp, d_ci, d_seeds, M, m, 11)
    assert ctx.check() == 0
    assert np.array_equal(walks.cpu().numpy(), w), "walks differ"
    del walks
    f_walks, f_off, f_ids, f_cnt = binding.sample_walks_rpe(ctx, d_rp, d_ci, d_seeds, M, m, 11)
    assert ctx.check() == 0
    assert np.array_equal(f_walks.cpu().numpy(), w), "fused: walks differ"
    assert_table_equal((f_off, f_ids, f_cnt), table, "fused rpe")
    # an entry that names no node: flagged, the walker stays where it is
    bad = ci.copy()
    bad[rp[7]] = n_leaves + 1 + 40
    walks = binding.sample_walks(ctx, d_rp, dev(bad), dev(np.full(seeds.size, 7, dtype=np.int32)),
                                 M, m, 11)
    assert ctx.check() == binding.DEV_BAD_GRAPH
    got = walks.cpu().numpy()
    assert ((got >= 0) & (got <= n_leaves)).all()
    stay = (got[:, :, 1] == 7)
    assert 0.2 < stay.mean() < 0.5                         # one of node 7's three entries


def random_graph_on_the_gpu(n_nodes, n_edges, active, seed):
    """CSR (row_ptr, col_idx) on the GPU: n_edges entries over `active` nodes spread over all ids."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    nodes = torch.randint(0, n_nodes, (active,), device="cuda", generator=g).unique()
    nodes[-1] = n_nodes - 1
    nodes = nodes.unique()
    deg = torch.zeros(n_nodes, dtype=torch.int64, device="cuda")
    deg[nodes] = n_edges // nodes.numel()
    deg[nodes[0]] += n_edges - int(deg.sum())
    rp = torch.zeros(n_nodes + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(deg, 0, out=rp[1:])
    ci = nodes[torch.randint(0, nodes.numel(), (n_edges,), device="cuda", generator=g)]
    return rp.int(), ci.int(), nodes.int()


@pytest.mark.parametrize("n_nodes,n_edges", [(1 << 27, 1 << 24), (1 << 23, (1 << 28) + 4321)])
def test_wide_edge_records(ctx, n_nodes, n_edges):
    # ids and row starts of 53 bits leave a packed record 11 bits for the degree, so the 16-byte
    # layout is used: few entries a node (rows looked up in groups), then many (from row_ptr)
    d_rp, d_ci, nodes = random_graph_on_the_gpu(n_nodes, n_edges, 1 << 18, n_nodes)
    rng = np.random.default_rng(1)
    M, m = 128, 15
    S = 4 * n_edges // (M * (m - 1)) + 5                   # enough steps to make the records
    d_seeds = nodes[torch.randint(0, nodes.numel(), (S,), device="cuda")].contiguous()
    lonely = S // 3
    d_seeds[lonely] = 12345 if int(d_rp[12346]) == int(d_rp[12345]) else 12346    # a node without neighbours
    walks = binding.sample_walks(ctx, d_rp, d_ci, d_seeds, M, m, 7)
    assert ctx.check() == 0
    # the walks of the same seeds without records (too few steps for them), and the oracle's
    part = S // 2
    for at in (0, S - part):
        assert torch.equal(binding.sample_walks(ctx, d_rp, d_ci, d_seeds[at:at + part].contiguous(), M,
                                                m, 7), walks[at:at + part])
    some = np.unique(np.r_[rng.integers(0, S, size=200), lonely, S - 1])
    rp, ci = d_rp.cpu().numpy(), d_ci.cpu().numpy()
    pick = torch.from_numpy(some).cuda()
    assert np.array_equal(walks[pick].cpu().numpy(),
                          oracle.sample_walks(rp, ci, d_seeds[pick].cpu().numpy(), M, m, 7))
    del rp, ci, walks
    # entries that name no node: flagged on both paths, the same walks
    d_bad = d_ci.clone()
    d_bad[::1001] = n_nodes
    a = binding.sample_walks(ctx, d_rp, d_bad, d_seeds, M, m, 7)
    assert ctx.check() == binding.DEV_BAD_GRAPH
    b = binding.sample_walks(ctx, d_rp, d_bad, d_seeds[:part].contiguous(), M, m, 7)
    assert ctx.check() == binding.DEV_BAD_GRAPH
    assert torch.equal(a[:part], b)


@pytest.mark.parametrize("M,m", [(128, 15), (100, 4), (50, 4), (200, 3)])
def test_fused_kernels_over_wide_edge_records(ctx, M, m):
    # the table (with counts, and with RPE-IDs) of the fused kernel against the two calls
    n_nodes, n_edges, L = 1 << 27, 1 << 24, m + 1
    d_rp, d_ci, nodes = random_graph_on_the_gpu(n_nodes, n_edges, 1 << 14, 3)
    S = 4 * n_edges // (M * (m - 1)) + 5
    d_seeds = nodes[torch.randint(0, nodes.numel(), (S,), device="cuda")].contiguous()
    d_seeds[S // 2] = n_nodes                              # not a node
    walks = binding.sample_walks(ctx, d_rp, d_ci, d_seeds, M, m, 7)
    assert ctx.check() == binding.DEV_BAD_SEED
    off, ids, cnt = binding.build_rpe(ctx, walks, n_nodes)
    assert ctx.check() == binding.DEV_BAD_WALK
    f_walks, f_off, f_ids, f_cnt = binding.sample_walks_rpe(ctx, d_rp, d_ci, d_seeds, M, m, 7)
    assert ctx.check() == binding.DEV_BAD_SEED
    assert torch.equal(f_walks, walks) and torch.equal(f_off, off) and torch.equal(f_ids, ids)
    assert torch.equal(f_cnt.view(torch.int16), cnt.view(torch.int16))
    del f_ids, f_cnt
    T, code = binding.prune_rpe(ctx, cnt, cap_T=1 << 22)
    assert ctx.check() == 0
    total = ids.numel()
    i_ids, i_code = (torch.empty(total, dtype=torch.int32, device="cuda") for _ in range(2))
    i_T = torch.zeros((1 << 22, L), dtype=torch.int16, device="cuda").view(torch.uint16)
    rc, rows, n_T = binding.sample_walks_rpe_ids_raw(ctx, d_rp, d_ci, d_seeds, M, m, 7, f_walks, total,
                                                     off, i_ids, None, i_code, 1 << 22, i_T)
    assert rc == binding.OK and rows == total and n_T == T.shape[0]
    assert ctx.check() == binding.DEV_BAD_SEED
    assert torch.equal(f_walks, walks) and torch.equal(i_ids, ids) and torch.equal(i_code, code)
    assert torch.equal(i_T[:n_T].view(torch.int16), T.view(torch.int16))


def test_one_call_rpe_ids_capacity(ctx):
    # surel_sample_walks_rpe_ids with too little room: for the table, for the distinct vectors
    wl = synth.Workload("t", "rmat", 256, 900, 0.0, 20, 3, 0, 2, "uniform", graph_seed=3)
    rp, ci = synth.make_graph(wl)
    M, m, L = wl.M, wl.m, wl.m + 1
    seeds = np.arange(64, dtype=np.int32)
    w = oracle.sample_walks(rp, ci, seeds, M, m, 3)
    t_off, t_ids, t_cnt = oracle.build_rpe(w)
    want_T, want_code = oracle.prune_rpe(t_cnt)
    total, n_T = int(t_off[-1]), want_T.shape[0]
    d_rp, d_ci, d_seeds = dev(rp), dev(ci), dev(seeds)
    walks = torch.empty((64, M, L), dtype=torch.int32, device="cuda")
    off = torch.empty(65, dtype=torch.int64, device="cuda")
    ids = torch.full((total,), -7, dtype=torch.int32, device="cuda")
    code = torch.full((total,), -7, dtype=torch.int32, device="cuda")
    T = torch.zeros((n_T, L), dtype=torch.int16, device="cuda").view(torch.uint16)
    # exactly enough room for both
    rc, rows, got_T = binding.sample_walks_rpe_ids_raw(ctx, d_rp, d_ci, d_seeds, M, m, 3, walks,
                                                       total, off, ids, None, code, n_T, T)
    assert rc == binding.OK and rows == total and got_T == n_T and ctx.check() == 0
    assert np.array_equal(host_u16(T), want_T) and np.array_equal(code.cpu().numpy(), want_code)
    assert np.array_equal(ids.cpu().numpy(), t_ids) and np.array_equal(off.cpu().numpy(), t_off)
    # one distinct vector too many
    rc, rows, got_T = binding.sample_walks_rpe_ids_raw(ctx, d_rp, d_ci, d_seeds, M, m, 3, walks,
                                                       total, off, ids, None, code, n_T - 1, T)
    assert rc == binding.E_CAPACITY and rows == total and got_T == n_T
    assert ctx.check() == binding.DEV_CAPACITY
    # a table that is too small: complete offsets and walks, the totals reported, nothing
    # written at or past cap_rows
    cap = total // 2
    ids.fill_(-7)
    code.fill_(-7)
    rc, rows, got_T = binding.sample_walks_rpe_ids_raw(ctx, d_rp, d_ci, d_seeds, M, m, 3, walks,
                                                       cap, off, ids, None, code, n_T, T)
    assert rc == binding.E_CAPACITY and rows == total
    assert ctx.check() == binding.DEV_CAPACITY
    assert np.array_equal(off.cpu().numpy(), t_off) and np.array_equal(walks.cpu().numpy(), w)
    assert (ids.cpu().numpy()[cap:] == -7).all() and (code.cpu().numpy()[cap:] == -7).all()
    last = int(t_off[1:][t_off[1:] <= cap].max())
    assert np.array_equal(ids.cpu().numpy()[:last], t_ids[:last])
    # no seeds at all
    rc, rows, got_T = binding.sample_walks_rpe_ids_raw(ctx, d_rp, d_ci, d_seeds[:0], M, m, 3,
                                                       walks[:0], 0, off[:1], ids, None, code, n_T, T)
    assert rc == binding.OK and rows == 0 and got_T == 0 and int(off[0]) == 0


@pytest.mark.parametrize("n_nodes, n_edges, malformed", [
    (65_535, 1 << 20, False), (65_536, 1 << 20, False), (1 << 18, (1 << 20) + 5, False),
    ((1 << 18) + 1, 1 << 20, False), (5 << 16, (1 << 20) + 1023, False), ((5 << 16) + 1, 1 << 20, False),
    (1, 1 << 20, False), (65_535, (1 << 20) - 1, False), (1500, (1 << 20) + 3, False),
    (65_535, 1 << 20, True), (200_000, 1 << 20, True), (30_000, (1 << 24) - 1, False),
    (30_000, 1 << 24, False)])
def test_short_edge_records(ctx, n_nodes, n_edges, malformed):
    # records that are ids of 1 to 19 bits, on both sides of every line between them and the packed
    # ones: uneven degrees, empty rows, a hub, entries and rows that are malformed
    rng = np.random.default_rng(n_nodes + n_edges)
    cuts = np.sort((rng.random(n_nodes - 1) ** 2 * (n_edges + 1)).astype(np.int64))
    rp = np.concatenate([[0], cuts, [n_edges]]).astype(np.int32)
    ci = rng.integers(0, n_nodes, size=n_edges).astype(np.int32)
    ci[-3:] = n_nodes - 1  # the last entries, whose words end behind the array
    M, m = 120, 5
    n_seeds = 9000 if n_edges < 1 << 23 else 34_953 * 4
    seeds = rng.integers(0, n_nodes, size=n_seeds).astype(np.int32)
    seeds[:9] = n_nodes - 1
    assert n_seeds * M * (m - 1) >= 4 * n_edges  # enough steps to make the records
    d_rp, d_ci, d_seeds = dev(rp), dev(ci), dev(seeds)
    if malformed:
        rp, ci = rp.copy(), ci.copy()
        rp[n_nodes // 3] = -5
        ci[::101] = n_nodes + rng.integers(0, 1000, size=ci[::101].size)
        ci[1::101] = n_nodes // 3
        d_rp, d_ci = dev(rp), dev(ci)
        w = binding.sample_walks(ctx, d_rp, d_ci, d_seeds, M, m, 3)
        assert ctx.check() == binding.DEV_BAD_GRAPH
        f = binding.sample_walks_rpe(ctx, d_rp, d_ci, d_seeds, M, m, 3)[0]
        assert ctx.check() == binding.DEV_BAD_GRAPH
        assert torch.equal(f, w) and bool(((w >= 0) & (w < n_nodes)).all())
        # a malformed row is never followed
        walks, lo, hi = w.cpu().numpy(), rp[:-1], rp[1:]
        at, moved = walks[:, :, :-1], walks[:, :, 1:] != walks[:, :, :-1]
        assert moved.any() and not (moved & ((lo[at] < 0) | (hi[at] < lo[at]))).any()
        return
    w = binding.sample_walks(ctx, d_rp, d_ci, d_seeds, M, m, 3)
    f = binding.sample_walks_rpe(ctx, d_rp, d_ci, d_seeds, M, m, 3)[0]
    assert ctx.check() == 0
    n = 4000
    assert torch.equal(f, w)
    assert np.array_equal(w[:n].cpu().numpy(), oracle.sample_walks(rp, ci, seeds[:n], M, m, 3))


@pytest.mark.parametrize("n_nodes", [1 << 17, (1 << 17) + 1])
@pytest.mark.parametrize("M", [128, 129])
def test_edge_records_of_walks_that_count_their_sets(ctx, n_nodes, M):
    # sets of about 640 nodes: the walks are those that are made without sizes, the sizes those of the walks
    m, n_edges, n_seeds = 5, 1 << 20, 9000
    rng = np.random.default_rng(n_nodes + M)
    cuts = np.sort((rng.random(n_nodes - 1) ** 2 * (n_edges + 1)).astype(np.int64))
    rp = np.concatenate([[0], cuts, [n_edges]]).astype(np.int32)
    ci = rng.integers(0, n_nodes, size=n_edges).astype(np.int32)
    seeds = rng.integers(0, n_nodes, size=n_seeds).astype(np.int32)
    sizes = torch.empty(n_seeds, dtype=torch.int32, device="cuda")
    w = binding.sample_walks(ctx, dev(rp), dev(ci), dev(seeds), M, m, 3, set_sizes=sizes)
    plain = binding.sample_walks(ctx, dev(rp), dev(ci), dev(seeds), M, m, 3)
    assert ctx.check() == 0
    assert torch.equal(w, plain)
    n = 500
    walks = w[:n].cpu().numpy()
    assert np.array_equal(walks, oracle.sample_walks(rp, ci, seeds[:n], M, m, 3))
    assert [len(np.unique(x)) for x in walks] == sizes[:n].cpu().tolist()


@pytest.mark.parametrize("M, m, n_seeds, n_nodes", [(1, 2, 4_200_000, 70_000), (4, 2, 1_100_000, 70_000),
                                                    (50, 4, 30_000, 3), (61, 9, 9000, 70_000),
                                                    (150, 4, 9400, 70_000), (200, 9, 3000, 70_000),
                                                    (200, 9, 3000, 330_000), (128, 15, 2400, 70_000),
                                                    (292, 6, 3000, 70_000), (500, 3, 3000, 70_000),
                                                    (682, 2, 6200, 70_000), (1024, 1, 3000, 70_000)])
def test_set_sizes_of_tables_that_fill_lds(ctx, M, m, n_seeds, n_nodes):
    # hash tables of any multiple of 64 slots, the smallest, the largest and the fullest among them (and of
    # powers of two where records are not short): every size against the sorted walks
    n_edges = 1 << 20
    rng = np.random.default_rng(M + m)
    cuts = np.sort(rng.integers(0, n_edges + 1, size=n_nodes - 1))
    rp = np.concatenate([[0], cuts, [n_edges]]).astype(np.int32)
    ci = rng.integers(0, n_nodes, size=n_edges).astype(np.int32)
    seeds = rng.integers(0, n_nodes, size=n_seeds).astype(np.int32)
    sizes = torch.empty(n_seeds, dtype=torch.int32, device="cuda")
    w = binding.sample_walks(ctx, dev(rp), dev(ci), dev(seeds), M, m, 3, set_sizes=sizes)
    assert ctx.check() == 0
    nodes = w.view(n_seeds, -1).sort(dim=1).values
    assert torch.equal(1 + (nodes[:, 1:] != nodes[:, :-1]).sum(dim=1).int(), sizes)
    n = 200
    assert np.array_equal(w[:n].cpu().numpy(), oracle.sample_walks(rp, ci, seeds[:n], M, m, 3))


@pytest.mark.parametrize("n_nodes, n_edges, M, m, n_seeds", [
    (5 << 16, 1 << 20, 150, 4, 9400), ((5 << 16) + 1, 1 << 20, 150, 4, 9400),
    (200_000, 1 << 20, 292, 6, 3000), (200_001, 1 << 20, 292, 6, 3000),
    (1 << 18, 12_000_000, 60, 5, 201_000), ((1 << 18) + 1, 11_999_999, 60, 5, 201_000),
    ((1 << 18) + 1, 12_000_000, 60, 5, 201_000)])
def test_edge_records_at_the_lines_between_their_forms(ctx, n_nodes, n_edges, M, m, n_seeds):
    # ids alone up to 5 * 2^16 nodes; up to 200,000 where sets of so many nodes are counted that few waves have
    # room; past 2^18 in walks + RPE only for fewer than 12,000,000 entries: the same walks in all of them
    assert n_seeds * M * (m - 1) >= 4 * n_edges  # enough steps to make the records
    rng = np.random.default_rng(n_nodes + n_edges)
    cuts = np.sort(rng.integers(0, n_edges + 1, size=n_nodes - 1))
    rp = np.concatenate([[0], cuts, [n_edges]]).astype(np.int32)
    ci = rng.integers(0, n_nodes, size=n_edges).astype(np.int32)
    seeds = rng.integers(0, n_nodes, size=n_seeds).astype(np.int32)
    d_rp, d_ci, d_seeds = dev(rp), dev(ci), dev(seeds)
    sizes = torch.empty(n_seeds, dtype=torch.int32, device="cuda")
    w = binding.sample_walks(ctx, d_rp, d_ci, d_seeds, M, m, 3, set_sizes=sizes)
    assert torch.equal(w, binding.sample_walks(ctx, d_rp, d_ci, d_seeds, M, m, 3))
    walks, off, _, _ = binding.sample_walks_rpe(ctx, d_rp, d_ci, d_seeds, M, m, 3)
    assert ctx.check() == 0
    assert torch.equal(w, walks) and torch.equal(off[1:] - off[:-1], sizes.long())
    nodes = w.view(n_seeds, -1).sort(dim=1).values
    assert torch.equal(1 + (nodes[:, 1:] != nodes[:, :-1]).sum(dim=1).int(), sizes)
    assert np.array_equal(w[:200].cpu().numpy(), oracle.sample_walks(rp, ci, seeds[:200], M, m, 3))


@pytest.mark.parametrize("n_nodes, malformed", [((1 << 18) - 1, False), (1 << 18, False),
                                           ((1 << 18) + 11, False), (1 << 18, True),
                                           ((5 << 18) - 1, False), (5 << 18, False),
                                           ((5 << 18) + 11, False), (5 << 18, True)])
def test_edge_records_of_grouped_rows(ctx, n_nodes, malformed):
    # from 5 * 2^18 nodes on rows are looked up in groups of 12: degrees at both sides of a byte's
    # range, an empty row, a hub, and rows behind them in their group and in the last, short one
    rng = np.random.default_rng(n_nodes)
    deg = rng.integers(0, 3, size=n_nodes)
    special = [0, 1, 253, 254, 255, 256, 0, 70_000]
    for at in (0, 11, 24, 12 * 2000 + 5, n_nodes - 9):
        deg[at:at + 8] = special[:min(8, n_nodes - at)]
    rp = np.zeros(n_nodes + 1, dtype=np.int64)
    np.cumsum(deg, out=rp[1:])
    # half of the neighbours are nodes near the special rows
    near = np.concatenate([np.arange(max(at - 3, 0), min(at + 30, n_nodes))
                           for at in (0, 11, 24, 12 * 2000 + 5, n_nodes - 9)])
    ci = rng.integers(0, n_nodes, size=int(rp[-1]))
    ci[::2] = rng.choice(near, size=ci[::2].size)
    seeds = rng.integers(0, n_nodes, size=40_000 if n_nodes < 1 << 19 else 60_000).astype(np.int32)
    seeds[::4] = rng.choice(near, size=seeds[::4].size)
    M, m = 60, 3
    rp, ci = rp.astype(np.int32), ci.astype(np.int32)
    assert seeds.size * M * (m - 1) >= 4 * ci.size         # enough steps to make the records
    if malformed:                                               # a malformed row: flagged, never followed
        rp[12 * 4000 + 3] = -7
        near_bad = np.arange(12 * 4000, 12 * 4001, dtype=np.int32)
        ci[1::64] = rng.choice(near_bad, size=ci[1::64].size)
        walks = binding.sample_walks(ctx, dev(rp), dev(ci), dev(seeds), M, m, 3).cpu().numpy()
        assert ctx.check() == binding.DEV_BAD_GRAPH
        assert ((walks >= 0) & (walks < n_nodes)).all()
        good = rp[:-1][walks[:, :, :-1]], rp[1:][walks[:, :, :-1]]
        moved = walks[:, :, 1:] != walks[:, :, :-1]
        bad_row = (good[0] < 0) | (good[1] < good[0])
        assert not (moved & bad_row).any()
        return
    walks = binding.sample_walks(ctx, dev(rp), dev(ci), dev(seeds), M, m, 3)
    assert ctx.check() == 0
    assert np.array_equal(walks.cpu().numpy(), oracle.sample_walks(rp, ci, seeds, M, m, 3))
