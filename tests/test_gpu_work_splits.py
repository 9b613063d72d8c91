"""Kernels whose work split has edges of its own, at the sizes where a split can go wrong, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import synth
from tests.test_gpu_parity import _expected_sampler_traffic

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import paper_2503_01281_amd as dci
    from tests import gpu_util as gu
    return dict(dci=dci, gu=gu, ctx=dci.Context(0))


# The list copy of the adjacency cache takes shares of 4,096 elements and stages at most 2,048 lists of a share at a time:
# one list over many shares, shares made of thousands of empty lists, lists that begin or end on a share's edge.
@pytest.mark.parametrize("lengths", [[20_001] + [0] * 5_000 + [1, 4_095, 4_096, 4_097], [1] * 4_097 + [0] * 2_050 + [3] * 700,
                                     [4_096, 8_192, 0, 1], [0] * 6_000 + [5]])
@pytest.mark.parametrize("share", [0.999, 0.4])
def test_list_copy_of_the_adjacency_cache(env, lengths, share):
    dci, gu, ctx = env["dci"], env["gu"], env["ctx"]
    rng = np.random.default_rng(len(lengths))
    indptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    N, E = len(lengths), int(indptr[-1])
    indices = rng.integers(0, N, E).astype(np.int64)
    count = np.arange(N, 0, -1).astype(np.uint32) if lengths[0] else rng.integers(0, 9, N).astype(np.uint32)
    c_adj = int(share * 8 * (N + 1 + E))
    remap, c_indptr, c_indices = oracle.fill_adj(indptr, indices, count, c_adj)
    g = gu.make_graph(indptr, indices, np.zeros((N, 1), dtype=np.float32))
    cache = dci.dci_fill_caches(ctx, g, gu.dev(np.zeros(N, dtype=np.int32)), gu.dev(count.view(np.int32)), c_adj, 1, 0,
                                dci.DCI_FILL_STRICT_SPLIT)
    K, M = cache.adj_nodes, cache.adj_edges
    assert (K, M) == (len(c_indptr) - 1, len(c_indices))
    assert np.array_equal(cache.adj_remap.cpu().numpy(), remap)
    words = cache.buf[cache.buf_offset:cache.buf_offset + 8 * (K + 1 + M)].view(torch.int64).cpu().numpy()
    assert np.array_equal(words[:K + 1], c_indptr) and np.array_equal(words[K + 1:], c_indices)


# The totals of the counters: fewer nodes than one workgroup's lanes, a remainder behind whole strides, and counters whose
# sum needs more than 32 bits (the paper's rule compares count * N with it).
@pytest.mark.parametrize("N", [1, 255, 1_025, 70_001])
def test_counter_totals_decide_the_feature_rows(env, N):
    dci, gu, ctx = env["dci"], env["gu"], env["ctx"]
    rng = np.random.default_rng(N)
    count = rng.integers(0, 2**32 - 1, N, dtype=np.uint32)
    feat = rng.standard_normal((N, 3)).astype(np.float32)
    g = gu.make_graph(np.minimum(np.arange(N + 1), 1).astype(np.int64), np.zeros(1, dtype=np.int64), feat)
    for policy in (0, 1):
        remap, rows, k = oracle.fill_feat(count, feat, 12 * (N // 3 + 1), policy)
        cache = dci.dci_fill_caches(ctx, g, gu.dev(count.view(np.int32)), gu.dev(np.zeros(N, dtype=np.int32)), 12 * (N // 3 + 1), 0, 1,
                                    policy | dci.DCI_FILL_STRICT_SPLIT)
        assert cache.feat_rows == k and np.array_equal(cache.feat_remap.cpu().numpy(), remap)
        got = cache.buf[cache.buf_offset:cache.buf_offset + cache.feat_bytes].view(torch.float32).cpu().numpy()
        assert np.array_equal(got.reshape(k, 3), rows)


# The sampler's node table is direct up to four nodes of the graph per node of the batch's bound, and hashed beyond: both sides
# of that line (768 nodes' bound; the smallest table, of 1,024 words), sizes that leave the cleared region a remainder, the
# first and last node ids, duplicate seeds and lists that repeat a hub.
@pytest.mark.parametrize("N,n_seeds", [(1, 5), (3, 2), (2_047, 3), (2_048, 3), (2_049, 3), (3_071, 64), (3_072, 64), (3_073, 64)])
def test_node_table_direct_and_hashed(env, N, n_seeds):
    dci, gu, ctx = env["dci"], env["gu"], env["ctx"]
    rng = np.random.default_rng(N)
    degree = rng.integers(0, 9, N)
    indptr = np.concatenate([[0], np.cumsum(degree)]).astype(np.int64)
    indices = np.where(rng.random(indptr[-1]) < 0.5, N - 1, rng.integers(0, N, indptr[-1])).astype(np.int64)
    seeds = rng.integers(0, N, n_seeds).astype(np.int64)
    seeds[0], seeds[-1] = N - 1, 0
    g = gu.make_graph(indptr, indices, None)
    blk = dci.Blocks(ctx, N, n_seeds, (3, 2))
    for batch in range(2):  # the second batch meets what the first left in the table
        for sample in (dci.dci_sample_khop, dci.dci_sample_khop_static):
            sample(ctx, g, None, gu.dev(seeds), batch, (3, 2), 7, blk)
            gu.assert_blocks_equal(gu.blocks_to_host(ctx, blk), oracle.sample_khop(indptr, indices, seeds, batch, (3, 2), 7))


# Floyd's chain over the slots of a lane group: fan-outs at the edges of the groups and between them, lists one longer than
# the fan-out (where collisions are the rule) and long ones.
@pytest.mark.parametrize("fanout", [1, 2, 4, 5, 6, 8, 9, 16, 17, 31, 32, 33, 62, 64])
def test_draw_chain_at_the_edges_of_its_steps(env, fanout):
    dci, gu, ctx = env["dci"], env["gu"], env["ctx"]
    N = 200
    rng = np.random.default_rng(fanout)
    degree = rng.choice([fanout - 1, fanout, fanout + 1, fanout + 2, 5 * fanout], N)
    indptr = np.concatenate([[0], np.cumsum(degree)]).astype(np.int64)
    indices = rng.integers(0, N, indptr[-1]).astype(np.int64)
    seeds = rng.permutation(N)[:101].astype(np.int64)
    g = gu.make_graph(indptr, indices, None)
    blk = dci.Blocks(ctx, N, len(seeds), (fanout,))
    dci.dci_sample_khop(ctx, g, None, gu.dev(seeds), 3, (fanout,), 11, blk)
    gu.assert_blocks_equal(gu.blocks_to_host(ctx, blk), oracle.sample_khop(indptr, indices, seeds, 3, (fanout,), 11))


# Tiles of the frontier scan: one row, a whole tile and one more, the last count of tiles that are numbered by their workgroup and the first
# with tickets (16 / 17), eight, and the line where a lane group takes two rows (200 / 201 tiles), for each width of a lane group.  With one
# hop, which is always scanned, and with another one behind it, where few rows of the first are one workgroup's (k_first_hops).
@pytest.mark.parametrize("fanout,rows_per_tile", [(2, 64), (9, 32), (17, 16), (33, 8)])
@pytest.mark.parametrize("tiles", [0, 1, 8, 16, 200])
@pytest.mark.parametrize("hashed", [False, True])
def test_tiles_of_the_frontier_scan(env, fanout, rows_per_tile, tiles, hashed):
    dci, gu, ctx = env["dci"], env["gu"], env["ctx"]
    N = 2_000_000 if hashed else 16_000
    rng = np.random.default_rng(fanout + tiles)
    degree = np.zeros(N, dtype=np.int64)
    degree[:16_000] = rng.integers(0, 2 * fanout, 16_000)
    indptr = np.concatenate([[0], np.cumsum(degree)]).astype(np.int64)
    indices = rng.integers(0, 16_000, indptr[-1]).astype(np.int64)
    g = gu.make_graph(indptr, indices, None, on_device=True)
    for extra in (0, 1):
        n = max(1, tiles * rows_per_tile) + extra
        seeds = rng.permutation(16_000)[:n].astype(np.int64)
        for fanouts in ((fanout,), (fanout, 2)):
            blk = dci.Blocks(ctx, N, n, fanouts)
            stats = gu.new_stats()
            ctx.timing_enable(["relabel"])
            dci.dci_sample_khop(ctx, g, None, gu.dev(seeds), extra, fanouts, 5, blk, stats)
            scans = ctx.timing_read()["relabel"][1]
            ctx.timing_enable([])
            assert scans == len(fanouts) - _first_hops(dci, N, n, fanouts)
            got = gu.blocks_to_host(ctx, blk)
            gu.assert_blocks_equal(got, oracle.sample_khop(indptr, indices, seeds, extra, fanouts, 5))
            s = gu.stats_dict(ctx, stats)
            assert s["edges_sampled"] == sum(got["n_edges"]) == s["adj_edge_misses"] and s["adj_node_misses"] == sum(got["n_nodes"][:-1])


def _first_hops(dci, N, n_seeds, fanouts):
    """Hops that one workgroup makes: from the first one on, all but the last at most, while rows (by their bound) times the widest lane
    group so far are 1,536 or fewer."""
    n = group = 0
    for rows, f in zip(dci.blocks_bounds(N, n_seeds, fanouts)[0], fanouts[:-1]):
        group = max(group, next(g for g in (8, 16, 32, 64) if f <= g))
        if rows * group > 1536:
            break
        n += 1
    return n


# Batches whose first hops are one kernel: the last number of seeds and the first beyond it for each width of a lane group (1,536 slots: 192
# rows of 8, ... 24 of 64), two and three such hops, with the hop behind them in the same batch; every kind of list (cached, not, in part).
@pytest.mark.parametrize("n_seeds,fanouts", [(1, (1, 1)), (192, (8, 3)), (193, (8, 3)), (96, (9, 2)), (97, (9, 2)), (48, (17, 2)), (49, (32, 1)),
                                             (24, (64, 2)), (25, (33, 2)), (16, (5, 10, 3)), (17, (5, 10, 3)), (5, (3, 3, 3, 2)), (3, (2, 40, 2)),
                                             (127, (2, 4, 8))])
@pytest.mark.parametrize("hashed", [False, True])
def test_first_hops_of_small_batches(env, n_seeds, fanouts, hashed):
    dci, gu, ctx = env["dci"], env["gu"], env["ctx"]
    N = 400_000 if hashed else 1_500
    rng = np.random.default_rng(n_seeds)
    degree = np.zeros(N, dtype=np.int64)
    degree[:1_500] = rng.integers(0, 2 * max(fanouts) + 3, 1_500)
    degree[7] = 500  # in part in the cache
    indptr = np.concatenate([[0], np.cumsum(degree)]).astype(np.int64)
    E = int(indptr[-1])
    indices = np.where(rng.random(E) < 0.1, rng.integers(0, 9, E), rng.integers(0, 1_500, E)).astype(np.int64)
    cached = np.sort(rng.permutation(np.arange(8, 1_500))[:600])
    remap = np.full(N, -1, dtype=np.int32)
    remap[cached], remap[7] = np.arange(600), 600
    lists = [indices[indptr[v]:indptr[v + 1]] for v in cached] + [indices[indptr[7]:indptr[7] + 200]]
    c_indptr = np.concatenate([[0], np.cumsum([len(x) for x in lists])]).astype(np.int64)
    cache = gu.upload_cache(remap, c_indptr, np.concatenate(lists), np.full(N, -1), np.zeros((0, 1), dtype=np.float32), 7, 500)
    g = gu.make_graph(indptr, indices, None)
    blk = dci.Blocks(ctx, N, n_seeds, fanouts)
    for batch in range(2):
        seeds = rng.permutation(1_500)[:n_seeds].astype(np.int64)
        seeds[0] = 7
        want = oracle.sample_khop(indptr, indices, seeds, batch, fanouts, 3)
        stats, plain = gu.new_stats(), gu.new_stats()
        ctx.timing_enable(["table_clear", "relabel"])
        dci.dci_sample_khop(ctx, g, cache, gu.dev(seeds), batch, fanouts, 3, blk, stats)
        launches = {k: v[1] for k, v in ctx.timing_read().items()}
        ctx.timing_enable([])
        n_first = _first_hops(dci, N, n_seeds, fanouts)
        assert (launches["table_clear"], launches["relabel"]) == (n_first == 0, len(fanouts) - n_first)
        gu.assert_blocks_equal(gu.blocks_to_host(ctx, blk), want)
        st, n_edges = gu.stats_dict(ctx, stats), int(sum(want.n_edges))
        rows = np.concatenate([want.nodes[:int(want.n_nodes[h])] for h in range(len(fanouts))])
        edges = np.concatenate([np.diff(want.blk_indptr[h]) for h in range(len(fanouts))])
        whole = (remap[rows] >= 0) & (rows != 7)
        assert st["adj_node_hits"] == (remap[rows] >= 0).sum() and st["adj_node_misses"] == (remap[rows] < 0).sum()
        assert edges[whole].sum() <= st["adj_edge_hits"] <= edges[whole].sum() + edges[rows == 7].sum()
        assert st["adj_edge_hits"] + st["adj_edge_misses"] == st["edges_sampled"] == n_edges and st["input_nodes"] == len(want.nodes)
        dci.dci_sample_khop_static(ctx, g, None, gu.dev(seeds), batch, fanouts, 3, blk, plain)
        gu.assert_blocks_equal(gu.blocks_to_host(ctx, blk), want)
        st = gu.stats_dict(ctx, plain)
        none = np.full(N, -1)
        assert (st["bytes_hbm"], st["bytes_host"], st["lines_bounds"], st["lines_ids"]) == _expected_sampler_traffic(
            want, fanouts, indptr, none, g.indptr.data_ptr(), g.indices.data_ptr())
    seeds = rng.permutation(1_500)[:2 * n_seeds + 1].astype(np.int64)
    feat, adj = (torch.zeros(N, dtype=torch.int32, device="cuda") for _ in range(2))
    edge = torch.zeros(E, dtype=torch.int32, device="cuda")
    dci.dci_presample_count(ctx, g, None, gu.dev(seeds), n_seeds, 0, 3, 9, fanouts, 3, feat, adj, edge)
    ctx.sync()
    f, a, e, _ = oracle.presample_count(indptr, indices, seeds, n_seeds, 3, fanouts, 3, 9)
    for got, counted in ((feat, f), (adj, a), (edge, e)):
        assert np.array_equal(got.cpu().numpy().view(np.uint32), counted)


@pytest.mark.parametrize("n_seeds,fanouts,n_first", [(30, (3, 2), 1), (20, (5, 10, 3), 1), (16, (5, 10, 3), 2), (300, (5, 3, 2), 0)])
def test_void_batch_behind_the_first_hops(env, n_seeds, fanouts, n_first):
    """A tile gives up (forced from the host; every kernel still ends at once) in the first hop behind those that are one kernel."""
    dci, gu = env["dci"], env["gu"]
    N = 3_000
    rng = np.random.default_rng(n_seeds)
    indptr = np.concatenate([[0], np.cumsum(rng.integers(1, 30, N))]).astype(np.int64)
    indices = rng.integers(0, N, indptr[-1]).astype(np.int64)
    g, ctx = gu.make_graph(indptr, indices, None), dci.Context(0)
    seeds = rng.permutation(N)[:n_seeds].astype(np.int64)
    blk, stats = dci.Blocks(ctx, N, n_seeds, fanouts), gu.new_stats()
    ctx.set_option(dci.DCI_OPT_RELABEL_SPIN_LIMIT, 200)
    for first in (1, 40):  # 40: beyond every frontier
        ctx.set_option(dci.DCI_OPT_TEST_RELABEL_FIRST_TICKET, first)
        ctx.timing_enable(["table_clear", "relabel"])
        dci.dci_sample_khop(ctx, g, None, gu.dev(seeds), 0, fanouts, 7, blk, stats)
        with pytest.raises(dci.DciError) as e:
            ctx.sync()
        assert e.value.code == -3 and "relabel scan timed out" in str(e.value)
        launches = {k: v[1] for k, v in ctx.timing_read().items()}
        ctx.timing_enable([])
        assert (launches["table_clear"], launches["relabel"]) == (n_first == 0, len(fanouts) - n_first)
        assert blk.counts.cpu().numpy().tolist() == [0] * 17 and blk.counts_host.numpy().tolist() == [0] * 17 and not stats.any()
    ctx.set_option(dci.DCI_OPT_TEST_RELABEL_FIRST_TICKET, 0)
    dci.dci_sample_khop(ctx, g, None, gu.dev(seeds), 0, fanouts, 7, blk, stats)
    gu.assert_blocks_equal(gu.blocks_to_host(ctx, blk), oracle.sample_khop(indptr, indices, seeds, 0, fanouts, 7))


# The selective gather's rounds of 32 to 256 looked-up rows to a workgroup, which follow from how many rows there are for its workgroups:
# a single row, a few, many; some cached, none, all.
@pytest.mark.parametrize("n", [1, 31, 33, 2_000, 150_000, 300_000, 600_000])
@pytest.mark.parametrize("share", [0.3, None, 1.0])
def test_rounds_of_the_selective_gather(env, n, share):
    dci, gu, ctx = env["dci"], env["gu"], env["ctx"]
    F, n_dense = 5, (n + 6) // 7
    g_ = torch.Generator().manual_seed(n)
    feat = torch.randn(n, F, generator=g_)
    g = dci.Graph(torch.zeros(n + 1, dtype=torch.int64).cuda(), torch.zeros(1, dtype=torch.int64).cuda(), feat.cuda())
    ids, remap, cache = torch.randperm(n, generator=g_), torch.full((n,), -1, dtype=torch.int32), None
    if share is not None:
        rows = torch.randperm(n, generator=g_)[:max(1, int(n * share))]
        remap[rows] = torch.arange(len(rows), dtype=torch.int32)
        cache = dci.Cache.from_arrays(torch.full((n,), -1, dtype=torch.int32).cuda(), torch.zeros(1, dtype=torch.int64).cuda(),
                                      torch.zeros(0, dtype=torch.int64).cuda(), remap.cuda(), feat[rows].cuda())
    blk = dci.Blocks(ctx, n, n_dense, (6,))
    blk.counts.zero_()
    blk.counts[0], blk.counts[1] = n_dense, n
    blk.nodes[:n] = ids.cuda()
    blk.blk_indptr[0].zero_()
    x = torch.full((max(n, blk.cap_nodes[1]), F), -7.0, device="cuda")
    w, b = torch.zeros(F, 4, device="cuda"), torch.zeros(4, device="cuda")
    y = torch.empty(blk.cap_nodes[0], 4, device="cuda")
    stats = gu.new_stats()
    dci.dci_gather_forward(ctx, g, cache, blk, x, 0, [w], [w], [b], y, stats)
    hit = remap[ids] >= 0
    st = gu.stats_dict(ctx, stats)
    copied = ~hit | (torch.arange(n) < n_dense)
    assert (st["feat_hits"], st["feat_misses"], st["rows_copied"]) == (int(hit.sum()), int((~hit).sum()), int(copied.sum()))
    got = x[:n].cpu()
    assert torch.equal(got[copied], feat[ids][copied]) and bool((got[~copied] == -7.0).all())
