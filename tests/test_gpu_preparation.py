"""Pre-sampling and the fill of the caches at the edges of how their work is cut up and handed back, against the oracle."""
import ctypes as C

import numpy as np
import pytest
import torch

import oracle

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
