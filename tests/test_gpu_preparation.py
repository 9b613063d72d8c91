"""Pre-sampling and the fill of the caches at the edges of how their work is cut up and handed back, against the oracle."""
import ctypes as C

import numpy as np
import pytest
import torch

import oracle
from tests.test_gpu_parity import _expected_sampler_traffic

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import paper_2503_01281_amd as dci
    from tests import gpu_util as gu
    return dict(dci=dci, gu=gu, ctx=dci.Context(0))


# A workspace that holds the node part of the element-granular fill and not its lists: the call fails after the copy of the
# feature rows (100 MB over the host link, milliseconds) has been enqueued, and must not return before it is over.
def test_failed_fill_leaves_the_stream_idle(env):
    dci, gu = env["dci"], env["gu"]
    N, F = 100_000, 256
    g = gu.make_graph(np.arange(N + 1, dtype=np.int64), np.zeros(N, dtype=np.int64), np.ones((N, F), dtype=np.float32))
    count = torch.ones(N, dtype=torch.int32, device="cuda")
    lib = dci.load_library()
    ctx = dci.Context(0)
    ws = torch.empty(lib.dci_fill_workspace_bytes(N) + 256, dtype=torch.uint8, device="cuda")
    ctx.check(lib.dci_set_workspace(ctx.handle, ws.data_ptr() + (-ws.data_ptr()) % 256, ws.numel() - 256))
    budget = 4 * N * F + 8 * N
    buf = torch.zeros(budget + 512, dtype=torch.uint8, device="cuda")
    remaps = torch.empty(2, N, dtype=torch.int32, device="cuda")
    out = (C.c_char * 256)()
    rc = lib.dci_fill_caches(ctx.handle, C.byref(g.c), count.data_ptr(), count.data_ptr(), count.data_ptr(), budget, 8 * N, 4 * N * F,
                             dci.DCI_FILL_STRICT_SPLIT | dci.DCI_FILL_ADJ_ELEMENTS, buf.data_ptr() + (-buf.data_ptr()) % 256,
                             remaps[0].data_ptr(), remaps[1].data_ptr(), g.indices.data_ptr(), out)
    assert torch.cuda.current_stream().query()
    assert rc == -2 and "element-granular fill" in lib.dci_last_error(ctx.handle).decode()


def fill_adjacency(env, indptr, indices, count, c_adj):
    dci, gu, ctx = env["dci"], env["gu"], env["ctx"]
    N = len(indptr) - 1
    g = gu.make_graph(indptr, indices, np.zeros((N, 1), dtype=np.float32), on_device=True)
    zeros, count = gu.dev(np.zeros(N, dtype=np.int32)), gu.dev(count.view(np.int32))
    ms = []
    for _ in range(3):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        cache = dci.dci_fill_caches(ctx, g, zeros, count, c_adj, 1, 0, dci.DCI_FILL_STRICT_SPLIT)
        b.record()
        b.synchronize()
        ms.append(a.elapsed_time(b))
    return cache, min(ms)


# Nodes without neighbours between two lists, all of them cached.  The copy of the lists shares the slots out as well as
# the elements: by elements alone one workgroup walks through all of the empty slots (a fill of 14.4 ms); the same fill with a
# budget for a few nodes takes 0.3 ms, and the 6 M slots add their list bounds and remap, 0.2 ms.
def test_run_of_empty_lists_is_shared_out(env):
    N = 6_000_000
    lengths = np.zeros(N, dtype=np.int64)
    lengths[[0, 1_000_000, N - 2, N - 1]] = 5_000, 1, 3_000, 1
    indptr = np.concatenate([[0], np.cumsum(lengths)])
    indices = np.random.default_rng(0).integers(0, N, int(indptr[-1]))
    count = np.zeros(N, dtype=np.uint32)
    c_adj = 8 * (N + 8_001)  # all but the last node
    cache, ms = fill_adjacency(env, indptr, indices, count, c_adj)
    remap, c_indptr, c_indices = oracle.fill_adj(indptr, indices, count, c_adj)
    K, M = cache.adj_nodes, cache.adj_edges
    assert (K, M) == (N - 1, 8_001) == (len(c_indptr) - 1, len(c_indices))
    assert np.array_equal(cache.adj_remap.cpu().numpy(), remap)
    words = cache.buf[cache.buf_offset:cache.buf_offset + 8 * (K + 1 + M)].view(torch.int64).cpu().numpy()
    assert np.array_equal(words[:K + 1], c_indptr) and np.array_equal(words[K + 1:], c_indices)
    _, few = fill_adjacency(env, indptr, indices, count, 8 * 5_010)
    print(f"fill of {K} lists {ms:.2f} ms, of a few {few:.2f} ms")
    assert ms < 3 * few + 1


# The closing kernel of a pre-sampled batch counts the visits of the input nodes and is billed as that; a batch that is
# only sampled has none to count.
def test_visit_counting_has_its_timing_class(env):
    dci, gu = env["dci"], env["gu"]
    N, fanouts = 500, (3, 2)
    rng = np.random.default_rng(1)
    indptr = np.arange(0, 6 * N + 1, 6, dtype=np.int64)
    g = gu.make_graph(indptr, rng.integers(0, N, 6 * N), None)
    seeds = gu.dev(rng.permutation(N)[:100])
    ctx = dci.Context(0)
    counts = [torch.zeros(N, dtype=torch.int32, device="cuda") for _ in range(2)]
    ctx.timing_enable(["write_src", "count_nodes"])
    dci.dci_presample_count(ctx, g, None, seeds, 20, 0, 5, 0, fanouts, 7, *counts)
    t = ctx.timing_read()
    assert t["count_nodes"][1] == 5 and t["count_nodes"][0] > 0 and t["write_src"] == (0.0, 0)
    dci.dci_sample_khop(ctx, g, None, seeds, 0, fanouts, 7, dci.Blocks(ctx, N, 100, fanouts))
    t = ctx.timing_read()
    assert t["write_src"][1] == 1 and t["write_src"][0] > 0 and t["count_nodes"] == (0.0, 0)


# With features loaded, pre-sampling waits and folds the gather's statistics once per 16 batches: whole runs, one batch over
# them, a last run of one, and a last batch that is short; all statistics against the oracle's batches.
@pytest.mark.parametrize("n_batches", [1, 15, 16, 17, 33])
def test_presampling_over_its_runs_of_batches(env, n_batches):
    dci, gu = env["dci"], env["gu"]
    N, F, batch, fanouts = 900, 5, 7, (3, 2)
    rng = np.random.default_rng(n_batches)
    indptr = np.concatenate([[0], np.cumsum(rng.integers(0, 9, N))]).astype(np.int64)
    indices = rng.integers(0, N, int(indptr[-1])).astype(np.int64)
    feat = rng.standard_normal((N, F)).astype(np.float32)
    g = gu.make_graph(indptr, indices, feat)
    seeds = rng.permutation(N)[:batch * n_batches - 3].astype(np.int64)
    weight = rng.integers(0, 9, N).astype(np.uint32)
    adj_remap, c_indptr, c_indices = oracle.fill_adj(indptr, indices, weight, 4 * (N + len(indices)))
    feat_remap, rows, _ = oracle.fill_feat(weight, feat, 2 * F * N, 1)
    cache = gu.upload_cache(adj_remap, c_indptr, c_indices, feat_remap, rows)
    ctx, stats = dci.Context(0), gu.new_stats()  # (a new context: its events are made by this call)
    counts = [torch.zeros(N, dtype=torch.int32, device="cuda") for _ in range(2)]
    scratch = torch.zeros(dci.blocks_bounds(N, batch, fanouts)[0][-1], F, device="cuda")
    dci.dci_presample_count(ctx, g, cache, gu.dev(seeds), batch, 0, n_batches + 2, 50, fanouts, 7, *counts, feat_scratch=scratch,
                            stats=stats)
    st = gu.stats_dict(ctx, stats)
    want = [oracle.sample_khop(indptr, indices, seeds[b * batch:(b + 1) * batch], 50 + b, fanouts, 7) for b in range(n_batches)]
    traffic = [_expected_sampler_traffic(b, fanouts, indptr, adj_remap, g.indptr.data_ptr(), g.indices.data_ptr()) for b in want]
    n_in = sum(len(b.nodes) for b in want)
    hits = sum(int((feat_remap[b.nodes] >= 0).sum()) for b in want)
    assert 0 < hits < n_in
    assert (st["feat_hits"], st["feat_misses"], st["rows_copied"], st["input_nodes"]) == (hits, n_in - hits, n_in, n_in)
    assert st["edges_sampled"] == sum(int(b.n_edges.sum()) for b in want)
    assert (st["bytes_hbm"], st["bytes_host"]) == (sum(t[0] for t in traffic) + 4 * F * hits,
                                                   sum(t[1] for t in traffic) + 4 * F * (n_in - hits))
    assert (st["lines_bounds"], st["lines_ids"]) == (sum(t[2] for t in traffic), sum(t[3] for t in traffic))
    assert st["t_sample_ns"] > 0 and st["t_feature_ns"] > 0
    assert np.array_equal(scratch[:len(want[-1].nodes)].cpu().numpy(), feat[want[-1].nodes])
    f, a, _, _ = oracle.presample_count(indptr, indices, seeds, batch, n_batches, fanouts, 7, 50)
    assert all(np.array_equal(got.cpu().numpy().view(np.uint32), w) for got, w in zip(counts, (f, a)))


def test_presampling_reports_a_voided_batch_at_the_end_of_its_run(env):
    dci, gu = env["dci"], env["gu"]
    N, batch, fanouts = 900, 7, (3, 2)
    g = gu.make_graph(np.arange(N + 1, dtype=np.int64), np.arange(N, dtype=np.int64), np.ones((N, 2), dtype=np.float32))
    seeds = gu.dev(np.arange(20 * batch))
    ctx, stats = dci.Context(0), gu.new_stats()
    counts = [torch.zeros(N, dtype=torch.int32, device="cuda") for _ in range(2)]
    scratch = torch.zeros(dci.blocks_bounds(N, batch, fanouts)[0][-1], 2, device="cuda")
    ctx.set_option(dci.DCI_OPT_RELABEL_SPIN_LIMIT, 200)
    ctx.set_option(dci.DCI_OPT_TEST_RELABEL_FIRST_TICKET, 1)
    with pytest.raises(dci.DciError) as e:
        dci.dci_presample_count(ctx, g, None, seeds, batch, 0, 20, 0, fanouts, 7, *counts, feat_scratch=scratch, stats=stats)
    assert e.value.code == -3 and "relabel scan timed out" in str(e.value)
    ctx.sync()  # reported once
    assert not counts[0].any() and not stats.any()  # every batch was voided: no input node was visited
    ctx.set_option(dci.DCI_OPT_TEST_RELABEL_FIRST_TICKET, 0)
    dci.dci_presample_count(ctx, g, None, seeds, batch, 0, 20, 0, fanouts, 7, *counts, feat_scratch=scratch, stats=stats)
    assert gu.stats_dict(ctx, stats)["input_nodes"] == int(counts[0].sum()) > 0
