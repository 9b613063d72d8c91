"""The sampler's node table in its four layouts - hashed, and direct with one, two or four words per node - with everything a
batch can come with: caches, statistics, pre-sampling counters, HIP-graph replays and a voided batch; against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from tests.test_gpu_parity import _expected_sampler_traffic

pytestmark = pytest.mark.gpu

FANOUTS, N_SEEDS, RNG_SEED = (5, 3), 40, 7
# 40 seeds bound the batch at 960 nodes (740 for 700 nodes): a hashed table of 15,360 (11,840) bytes.  Direct is chosen at 4 bytes
# per node and less, and takes the most words per node that fit into those bytes.
LAYOUTS = {"hashed": 4_000, "direct": 3_000, "two words": 1_500, "four words": 700}


@pytest.fixture(scope="module", params=list(LAYOUTS))
def env(request):
    import paper_2503_01281_amd as dci
    from tests import gpu_util as gu
    N = LAYOUTS[request.param]
    rng = np.random.default_rng(N)
    indptr = np.concatenate([[0], np.cumsum(rng.integers(0, 13, N))]).astype(np.int64)
    E = int(indptr[-1])
    indices = np.where(rng.random(E) < 0.2, rng.integers(0, 9, E), rng.integers(0, N, E)).astype(np.int64)  # with hubs
    seeds = rng.permutation(N)[:4 * N_SEEDS].astype(np.int64)
    return dict(dci=dci, gu=gu, ctx=dci.Context(0), N=N, indptr=indptr, indices=indices, seeds=seeds,
                graph=gu.make_graph(indptr, indices, None))


def expected(e, seeds, batch):
    return oracle.sample_khop(e["indptr"], e["indices"], seeds, batch, FANOUTS, RNG_SEED)


def test_cache_and_statistics(env):
    dci, gu, ctx, g = (env[k] for k in ("dci", "gu", "ctx", "graph"))
    N, indptr, indices = env["N"], env["indptr"], env["indices"]
    count = np.random.default_rng(1).integers(0, 9, N).astype(np.uint32)
    remap, c_indptr, c_indices = oracle.fill_adj(indptr, indices, count, 4 * (N + len(indices)))
    cache = gu.upload_cache(remap, c_indptr, c_indices, np.full(N, -1), np.zeros((0, 1), dtype=np.float32))
    blk = dci.Blocks(ctx, N, N_SEEDS, FANOUTS)
    for batch in range(3):
        seeds, stats = env["seeds"][batch * N_SEEDS:(batch + 1) * N_SEEDS], gu.new_stats()
        want = expected(env, seeds, batch)
        dci.dci_sample_khop(ctx, g, cache, gu.dev(seeds), batch, FANOUTS, RNG_SEED, blk, stats)
        gu.assert_blocks_equal(gu.blocks_to_host(ctx, blk), want)
        st = gu.stats_dict(ctx, stats)
        traffic = _expected_sampler_traffic(want, FANOUTS, indptr, remap, g.indptr.data_ptr(), g.indices.data_ptr())
        assert (st["bytes_hbm"], st["bytes_host"], st["lines_bounds"], st["lines_ids"]) == traffic
        hit = [remap[want.nodes[:int(want.n_nodes[h])]] >= 0 for h in range(2)]
        edges = [np.diff(want.blk_indptr[h]) for h in range(2)]
        assert st["adj_node_hits"] == sum(int(m.sum()) for m in hit) > 0 and st["adj_node_misses"] > 0
        assert st["adj_edge_hits"] == sum(int(c[m].sum()) for c, m in zip(edges, hit))
        assert (st["edges_sampled"], st["input_nodes"]) == (sum(int(c.sum()) for c in edges), len(want.nodes))


def test_presampling_counters(env):
    dci, gu, ctx, g = (env[k] for k in ("dci", "gu", "ctx", "graph"))
    seeds = env["seeds"][:4 * N_SEEDS - 11]  # the last batch is short
    feat, adj = (torch.zeros(env["N"], dtype=torch.int32, device="cuda") for _ in range(2))
    edge = torch.zeros(max(len(env["indices"]), 1), dtype=torch.int32, device="cuda")
    dci.dci_presample_count(ctx, g, None, gu.dev(seeds), N_SEEDS, 0, 4, 1 << 31, FANOUTS, RNG_SEED, feat, adj, edge)
    ctx.sync()
    f, a, e, _ = oracle.presample_count(env["indptr"], env["indices"], seeds, N_SEEDS, 4, FANOUTS, RNG_SEED, 1 << 31)
    for got, want in ((feat, f), (adj, a), (edge, e)):
        assert np.array_equal(got.cpu().numpy().view(np.uint32)[:len(want)], want)


def test_replays_from_a_hip_graph(env):
    dci, gu, g, N = (env[k] for k in ("dci", "gu", "graph", "N"))
    side = torch.cuda.Stream()
    ctx = dci.Context(0, stream=side)
    with torch.cuda.stream(side):
        blk = dci.Blocks(ctx, N, N_SEEDS, FANOUTS)
        all_seeds = gu.dev(env["seeds"])
        seeds = all_seeds[:N_SEEDS].clone()
        dci.dci_sample_khop(ctx, g, None, seeds, 3, FANOUTS, RNG_SEED, blk)  # sizes the workspace before the capture
        ctx.sync()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            dci.dci_sample_khop(ctx, g, None, seeds, 3, FANOUTS, RNG_SEED, blk)
        for r in (0, 1, 2, 0, 3):
            seeds.copy_(all_seeds[r * N_SEEDS:(r + 1) * N_SEEDS])
            want = expected(env, env["seeds"][r * N_SEEDS:(r + 1) * N_SEEDS], 3)
            for step in (lambda: dci.dci_sample_khop(ctx, g, None, seeds, 3, FANOUTS, RNG_SEED, blk), graph.replay):
                for t in [blk.nodes, blk.counts] + blk.blk_indptr + blk.blk_src:
                    t.fill_(-1)
                step()
                gu.assert_blocks_equal(gu.blocks_to_host(ctx, blk), want)


def test_voided_batch(env):
    dci, gu, g, N = (env[k] for k in ("dci", "gu", "graph", "N"))
    ctx = dci.Context(0)
    blk, stats = dci.Blocks(ctx, N, N_SEEDS, FANOUTS), gu.new_stats()
    seeds = env["seeds"][:N_SEEDS]
    ctx.set_option(dci.DCI_OPT_RELABEL_SPIN_LIMIT, 200)
    ctx.set_option(dci.DCI_OPT_TEST_RELABEL_FIRST_TICKET, 1)
    dci.dci_sample_khop(ctx, g, None, gu.dev(seeds), 0, FANOUTS, RNG_SEED, blk, stats)
    with pytest.raises(dci.DciError) as e:
        ctx.sync()
    assert e.value.code == -3 and blk.counts.cpu().numpy().tolist() == [0] * 17 and not stats.any()
    ctx.set_option(dci.DCI_OPT_TEST_RELABEL_FIRST_TICKET, 0)
    dci.dci_sample_khop(ctx, g, None, gu.dev(seeds), 0, FANOUTS, RNG_SEED, blk, stats)
    gu.assert_blocks_equal(gu.blocks_to_host(ctx, blk), expected(env, seeds, 0))


# A direct table is spread over at most 4 MB: both sides of the node counts at which it falls back to two words per node and to one.
@pytest.mark.parametrize("N", [262_144, 262_145, 524_288, 524_289])
def test_direct_table_at_the_edges_of_its_spread(N):
    import paper_2503_01281_amd as dci
    from tests import gpu_util as gu
    ctx, rng = dci.Context(0), np.random.default_rng(N)
    indptr = np.arange(0, 7 * N + 1, 7, dtype=np.int64)
    indices = rng.integers(0, N, 7 * N)
    seeds = rng.permutation(N)[:20_000].astype(np.int64)
    seeds[:2] = N - 1, 0
    g = gu.make_graph(indptr, indices, None)
    blk = dci.Blocks(ctx, N, len(seeds), (5, 10))
    dci.dci_sample_khop(ctx, g, None, gu.dev(seeds), 1, (5, 10), RNG_SEED, blk)
    gu.assert_blocks_equal(gu.blocks_to_host(ctx, blk), oracle.sample_khop(indptr, indices, seeds, 1, (5, 10), RNG_SEED))
