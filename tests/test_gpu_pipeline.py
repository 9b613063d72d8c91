"""dci_infer_batches: many batches with several in flight (one lane = context + stream + buffers).

Sixteen consecutive batches of the Tiny workload run on four lanes through partially filled caches (so the
hit and the miss routes of both the sampler and the gather are live), and every batch is compared with the
CPU oracle: blocks and gathered rows bit for bit, logits to 1e-4 of the batch's largest logit.  Blocks and
rows of a batch survive only until its lane takes the next one, so the sixteen batches are run twice: once
in a single call (all logits checked, and the blocks / rows of the last batch of every lane), once four at
a time with every lane's blocks and rows checked in between."""
import ctypes as C

import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu

B = 128          # 2,048 seeds -> 16 batches
N_LANES = 4


@pytest.fixture(scope="module")
def setup(tiny):
    import paper_2503_01281_amd as dci
    from tests import gpu_util as gu
    w = tiny["w"]
    ctx = dci.Context(0)
    g = gu.make_graph(tiny["indptr"], tiny["indices"], tiny["feat"])
    fc, ac, _, _ = oracle.presample_count(tiny["indptr"], tiny["indices"], tiny["seeds"], w.batch_size, w.n_presample,
                                          w.fanouts, w.rng_seed, w.presample_first_batch, with_edge_count=False)
    C_adj, C_feat = oracle.split(w.budget_bytes, 3, 7, w.num_nodes, w.num_edges, w.feat_dim)
    adj_remap, cp, ci = oracle.fill_adj(tiny["indptr"], tiny["indices"], ac, C_adj)
    feat_remap, fcache, k = oracle.fill_feat(fc, tiny["feat"], C_feat, 0)
    assert 0 < (adj_remap >= 0).sum() < w.num_nodes and 0 < k < w.num_nodes      # both caches partial
    cache = gu.upload_cache(adj_remap, cp, ci, feat_remap, fcache)
    weights = [[gu.dev(a) for a in tiny[key]] for key in ("w_self", "w_neigh", "bias")]
    lanes = [dci.Lane(g, B, w.fanouts, w.dims) for _ in range(N_LANES)]
    seeds_dev = gu.dev(tiny["seeds"])
    torch.cuda.synchronize()
    want = []
    for b in range(w.num_seeds // B):
        s = tiny["seeds"][b * B:(b + 1) * B]
        blk = oracle.sample_khop(tiny["indptr"], tiny["indices"], s, b, w.fanouts, w.rng_seed)
        x = oracle.gather(tiny["feat"], blk.nodes)
        want.append((blk, x))
    return dict(dci=dci, gu=gu, w=w, g=g, cache=cache, weights=weights, lanes=lanes, seeds=seeds_dev, want=want,
                adj_remap=adj_remap, feat_remap=feat_remap, tiny=tiny)


def _check_lane(gu, lane, blk_want, x_want):
    got = gu.blocks_to_host(lane.ctx, lane.blocks)
    gu.assert_blocks_equal(got, blk_want)
    assert lane.x[:len(blk_want.nodes)].cpu().numpy().tobytes() == x_want.tobytes()


def _check_logits(got, ref):
    assert np.abs(got - ref).max() <= 1e-4 * max(1.0, np.abs(ref).max())


@pytest.mark.parametrize("model", [0, 2])
def test_sixteen_batches_on_four_lanes(setup, model):
    dci, gu, w, g, cache, lanes, want, tiny = (setup[k] for k in ("dci", "gu", "w", "g", "cache", "lanes", "want", "tiny"))
    ws, wn, bs = setup["weights"]
    nb = len(want)
    assert nb == 16
    ref = [oracle.gnn_forward(model, blk, x, tiny["w_self"], tiny["w_neigh"], tiny["bias"]) for blk, x in want]
    logits = torch.full((w.num_seeds, w.classes), float("nan"), dtype=torch.float32, device="cuda")
    stats = gu.new_stats()
    torch.cuda.synchronize()

    # all sixteen in one call
    dci.dci_infer_batches(lanes, g, cache, setup["seeds"], B, 0, nb, w.fanouts, w.rng_seed, model,
                          None if model == 2 else ws, wn, bs, logits, stats)
    for ln in lanes:
        ln.ctx.sync()
    out = logits.cpu().numpy()
    for b in range(nb):
        _check_logits(out[b * B:(b + 1) * B], ref[b])
    for k, ln in enumerate(lanes):                       # lane k ran batches k, k+4, k+8, k+12
        _check_lane(gu, ln, *want[nb - N_LANES + k])
    st = {k: int(v) for k, v in zip(dci.STAT.keys(), stats.cpu().numpy())}
    assert st["edges_sampled"] == sum(int(blk.n_edges.sum()) for blk, _ in want)
    assert st["input_nodes"] == sum(len(blk.nodes) for blk, _ in want)
    hits = sum(int((setup["feat_remap"][blk.nodes] >= 0).sum()) for blk, _ in want)
    assert (st["feat_hits"], st["feat_misses"]) == (hits, st["input_nodes"] - hits)
    assert 0 < st["adj_edge_hits"] < st["edges_sampled"] and 0 < hits < st["input_nodes"]

    # four at a time, every lane's blocks and rows checked while they are still there
    logits.fill_(float("nan"))
    for first in range(0, nb, N_LANES):
        dci.dci_infer_batches(lanes, g, cache, setup["seeds"], B, first, N_LANES, w.fanouts, w.rng_seed, model,
                              None if model == 2 else ws, wn, bs, logits)
        for ln in lanes:
            ln.ctx.sync()
        for k, ln in enumerate(lanes):
            _check_lane(gu, ln, *want[first + k])
    out = logits.cpu().numpy()
    for b in range(nb):
        _check_logits(out[b * B:(b + 1) * B], ref[b])


def test_fused_input_lanes_give_the_same_logits(setup):
    """DCI_OPT_FUSED_INPUT on every lane: cached neighbour rows are read in place; logits of all sixteen batches
    against the oracle, blocks bit for bit, statistics as with the two-call route."""
    dci, gu, w, g, cache, lanes, want, tiny = (setup[k] for k in ("dci", "gu", "w", "g", "cache", "lanes", "want", "tiny"))
    ws, wn, bs = setup["weights"]
    nb = len(want)
    logits = torch.full((w.num_seeds, w.classes), float("nan"), dtype=torch.float32, device="cuda")
    stats = gu.new_stats()
    torch.cuda.synchronize()
    for ln in lanes:
        ln.ctx.set_option(dci.DCI_OPT_FUSED_INPUT, 1)
    try:
        dci.dci_infer_batches(lanes, g, cache, setup["seeds"], B, 0, nb, w.fanouts, w.rng_seed, 0, ws, wn, bs, logits, stats)
        for ln in lanes:
            ln.ctx.sync()
    finally:
        for ln in lanes:
            ln.ctx.set_option(dci.DCI_OPT_FUSED_INPUT, 0)
    out = logits.cpu().numpy()
    for b, (blk, x) in enumerate(want):
        _check_logits(out[b * B:(b + 1) * B], oracle.sage_forward(blk, x, tiny["w_self"], tiny["w_neigh"], tiny["bias"]))
    for k, ln in enumerate(lanes):
        gu.assert_blocks_equal(gu.blocks_to_host(ln.ctx, ln.blocks), want[nb - N_LANES + k][0])
    st = {k: int(v) for k, v in zip(dci.STAT.keys(), stats.cpu().numpy())}
    hits = sum(int((setup["feat_remap"][blk.nodes] >= 0).sum()) for blk, _ in want)
    assert (st["feat_hits"], st["feat_hits"] + st["feat_misses"]) == (hits, sum(len(blk.nodes) for blk, _ in want))


def test_ragged_last_batch_and_ranges(setup):
    """A seed list that ends inside a batch, a range that runs past the last batch, an empty range, one lane."""
    dci, gu, w, g, cache, lanes, tiny = (setup[k] for k in ("dci", "gu", "w", "g", "cache", "lanes", "tiny"))
    ws, wn, bs = setup["weights"]
    n = 5 * B + 37
    seeds = setup["seeds"][:n]
    logits = torch.full((n, w.classes), float("nan"), dtype=torch.float32, device="cuda")
    torch.cuda.synchronize()
    dci.dci_infer_batches(lanes[:3], g, cache, seeds, B, 2, 0, w.fanouts, w.rng_seed, 0, ws, wn, bs, logits)   # nothing
    dci.dci_infer_batches(lanes[:3], g, cache, seeds, B, 2, 100, w.fanouts, w.rng_seed, 0, ws, wn, bs, logits)  # 2..5
    dci.dci_infer_batches(lanes[3:], g, cache, seeds, B, 0, 2, w.fanouts, w.rng_seed, 0, ws, wn, bs, logits)    # 0, 1
    for ln in lanes:
        ln.ctx.sync()
    out = logits.cpu().numpy()
    assert not np.isnan(out).any()
    for b in range(6):
        s = tiny["seeds"][b * B:min(n, (b + 1) * B)]
        blk = oracle.sample_khop(tiny["indptr"], tiny["indices"], s, b, w.fanouts, w.rng_seed)
        ref = oracle.sage_forward(blk, oracle.gather(tiny["feat"], blk.nodes), tiny["w_self"], tiny["w_neigh"], tiny["bias"])
        _check_logits(out[b * B:b * B + len(s)], ref)
    # of the three lanes, lane 0 ran batches 2 and 5: it holds the ragged last batch (37 seeds)
    last = oracle.sample_khop(tiny["indptr"], tiny["indices"], tiny["seeds"][5 * B:n], 5, w.fanouts, w.rng_seed)
    assert last.n_nodes[0] == 37
    _check_lane(gu, lanes[0], last, oracle.gather(tiny["feat"], last.nodes))


def test_lanes_must_not_share(setup):
    dci, w, g, cache, lanes = (setup[k] for k in ("dci", "w", "g", "cache", "lanes"))
    ws, wn, bs = setup["weights"]
    logits = torch.empty(w.num_seeds, w.classes, dtype=torch.float32, device="cuda")
    with pytest.raises(dci.DciError) as e:
        dci.dci_infer_batches([lanes[0], lanes[0]], g, cache, setup["seeds"], B, 0, 2, w.fanouts, w.rng_seed, 0, ws, wn, bs,
                              logits)
    assert e.value.code == -1 and "share" in str(e.value)


@pytest.mark.parametrize("fused", [0, 1])
def test_batches_closed_beside_the_gather(setup, fused):
    """A batch is closed beside its gather where the workspace holds both stages' temporaries and no statistics are asked for: blocks, rows and
    logits bit for bit those of the stages in sequence (with statistics; with a workspace for one stage at a time)."""
    dci, gu, w, g, cache, want = (setup[k] for k in ("dci", "gu", "w", "g", "cache", "want"))
    ws, wn, bs = setup["weights"]
    got = []
    for way in ("beside", "statistics", "small workspace"):
        ln = dci.Lane(g, B, w.fanouts, w.dims)
        if way == "small workspace":
            caps = (C.c_int64 * dci.DCI_MAX_HOPS)(*(list(ln.blocks.cap_nodes[:w.n_hops]) + [0] * (dci.DCI_MAX_HOPS - w.n_hops)))
            lib, L = ln.ctx.lib, w.n_hops
            arr = lambda v: (C.c_int32 * len(v))(*v)
            need = max(lib.dci_sample_workspace_bytes(w.num_nodes, B, arr(w.fanouts), L),
                       lib.dci_gather_forward_workspace_bytes(ln.blocks.cap_nodes[L], caps, L, arr(w.dims)))
            small = torch.empty(need + 256, dtype=torch.uint8, device="cuda")
            assert lib.dci_set_workspace(ln.ctx.handle, (small.data_ptr() + 255) // 256 * 256, need) == 0
        ln.ctx.set_option(dci.DCI_OPT_FUSED_INPUT, fused)
        logits = torch.full((w.num_seeds, w.classes), float("nan"), dtype=torch.float32, device="cuda")
        ln.x.fill_(-5.0)
        torch.cuda.synchronize()
        ln.ctx.timing_enable(["write_src"])
        dci.dci_infer_batches([ln], g, cache, setup["seeds"], B, 3, 2, w.fanouts, w.rng_seed, 0, ws, wn, bs, logits,
                              gu.new_stats() if way == "statistics" else None)
        assert ln.ctx.timing_read()["write_src"][1] == (0 if way == "beside" else 2)
        gu.assert_blocks_equal(gu.blocks_to_host(ln.ctx, ln.blocks), want[4][0])
        got.append((logits[3 * B:5 * B].cpu().numpy().tobytes(), ln.x.cpu().numpy().tobytes()))
    assert got[0] == got[1] == got[2] and not np.isnan(np.frombuffer(got[0][0], dtype=np.float32)).any()


# Both kinds of node table, rows of 16, 8 and 4 bytes at a time, every row cached, some, none, the three models, rows read in place or
# gathered.
@pytest.mark.parametrize("hashed,F,cached,model,fused", [
    (False, 8, 0.4, 0, 1), (True, 8, 0.4, 0, 1), (True, 6, None, 1, 1), (True, 5, 1.0, 2, 1), (False, 6, 1.0, 1, 1), (False, 5, 0.4, 2, 1),
    (False, 5, None, 2, 0), (True, 6, 0.4, 0, 0), (True, 8, 1.0, 1, 0), (False, 8, None, 0, 0)])
def test_batches_closed_beside_every_form_of_the_gather(hashed, F, cached, model, fused):
    import paper_2503_01281_amd as dci
    from tests import gpu_util as gu
    used, fanouts, batch, n_batches = 4_000, (4, 3, 6), 301, 3
    N = 600_000 if hashed else used
    dims = (F, 12, 9, 7)
    rng = np.random.default_rng(F + model)
    degree = np.zeros(N, dtype=np.int64)
    degree[:used] = rng.integers(0, 11, used)
    indptr = np.concatenate([[0], np.cumsum(degree)]).astype(np.int64)
    indices = rng.integers(0, used, indptr[-1]).astype(np.int64)
    feat = rng.standard_normal((N, F)).astype(np.float32)
    g = gu.make_graph(indptr, indices, feat)
    cache = None
    if cached is not None:
        rows = np.sort(rng.permutation(N)[:int(cached * N)])
        remap = np.full(N, -1, dtype=np.int32)
        remap[rows] = np.arange(len(rows))
        cache = gu.upload_cache(np.full(N, -1), np.zeros(1), np.zeros(0), remap, feat[rows])
    seeds = rng.permutation(used)[:batch * n_batches - 50].astype(np.int64)
    pairs = list(zip(dims, dims[1:]))
    ws, wn = ([rng.uniform(-1, 1, p).astype(np.float32) for p in pairs] for _ in range(2))
    bs = [rng.uniform(-1, 1, p[1]).astype(np.float32) for p in pairs]
    out = []
    for stats in (None, gu.new_stats()):
        ln = dci.Lane(g, batch, fanouts, dims)
        ln.ctx.set_option(dci.DCI_OPT_FUSED_INPUT, fused)
        logits = torch.full((len(seeds), dims[-1]), float("nan"), dtype=torch.float32, device="cuda")
        ln.x.fill_(-5.0)
        seeds_dev, weights = gu.dev(seeds), [[gu.dev(a) for a in p] for p in (ws, wn, bs)]
        if model == 2:
            weights[0] = None
        torch.cuda.synchronize()
        ln.ctx.timing_enable(["write_src"])
        dci.dci_infer_batches([ln], g, cache, seeds_dev, batch, 0, n_batches, fanouts, 17, model, *weights, logits, stats)
        assert ln.ctx.timing_read()["write_src"][1] == (0 if stats is None else n_batches)
        blk = gu.blocks_to_host(ln.ctx, ln.blocks)
        gu.assert_blocks_equal(blk, oracle.sample_khop(indptr, indices, seeds[2 * batch:], 2, fanouts, 17))
        out.append((logits.cpu().numpy(), ln.x.cpu().numpy().tobytes()))
    assert out[0][0].tobytes() == out[1][0].tobytes() and out[0][1] == out[1][1]
    for b in range(n_batches):
        blk = oracle.sample_khop(indptr, indices, seeds[b * batch:(b + 1) * batch], b, fanouts, 17)
        _check_logits(out[0][0][b * batch:(b + 1) * batch], oracle.gnn_forward(model, blk, oracle.gather(feat, blk.nodes), ws, wn, bs))


@pytest.mark.parametrize("beyond", [0, 1])
def test_large_batches_of_gathered_rows_are_closed_by_a_kernel_of_their_own(beyond):
    """More than 512 slots of the last hop for every compute unit, by their bound; rows read in place are closed beside whatever the size."""
    import paper_2503_01281_amd as dci
    from tests import gpu_util as gu
    batch = torch.cuda.get_device_properties(0).multi_processor_count * 512 // 32 + beyond  # 4 rows of 8 slots to a seed
    N, F, fanouts, dims = 20_000, 5, (3, 8), (5, 6, 4)
    rng = np.random.default_rng(9)
    indptr = np.concatenate([[0], np.cumsum(rng.integers(0, 20, N))]).astype(np.int64)
    indices = rng.integers(0, N, indptr[-1]).astype(np.int64)
    feat = rng.standard_normal((N, F)).astype(np.float32)
    g = gu.make_graph(indptr, indices, feat, on_device=True)
    seeds = rng.permutation(N)[:batch].astype(np.int64)
    w = [rng.uniform(-1, 1, p).astype(np.float32) for p in zip(dims, dims[1:])]
    b = [np.zeros(n, dtype=np.float32) for n in dims[1:]]
    ln = dci.Lane(g, batch, fanouts, dims)
    seeds_dev, w_dev, b_dev = gu.dev(seeds), [gu.dev(a) for a in w], [gu.dev(a) for a in b]
    want = oracle.sample_khop(indptr, indices, seeds, 0, fanouts, 3)
    ref = oracle.gnn_forward(0, want, oracle.gather(feat, want.nodes), w, w, b)
    for fused in (0, 1):
        ln.ctx.set_option(dci.DCI_OPT_FUSED_INPUT, fused)
        logits = torch.full((batch, dims[-1]), float("nan"), dtype=torch.float32, device="cuda")
        torch.cuda.synchronize()
        ln.ctx.timing_enable(["write_src"])
        dci.dci_infer_batches([ln], g, None, seeds_dev, batch, 0, 1, fanouts, 3, 0, w_dev, w_dev, b_dev, logits)
        assert ln.ctx.timing_read()["write_src"][1] == (1 if beyond and not fused else 0)
        gu.assert_blocks_equal(gu.blocks_to_host(ln.ctx, ln.blocks), want)
        _check_logits(logits.cpu().numpy(), ref)


def test_a_lane_without_memory_for_both_stages_takes_room_for_one(setup, monkeypatch):
    dci, gu, w, g, want = (setup[k] for k in ("dci", "gu", "w", "g", "want"))
    ws, wn, bs = setup["weights"]
    asked, ensure = [], dci.Context.ensure_workspace

    def full(self, nbytes):
        asked.append(nbytes)
        if len(asked) == 1:
            raise torch.OutOfMemoryError("no room")
        ensure(self, nbytes)

    monkeypatch.setattr(dci.Context, "ensure_workspace", full)
    ln = dci.Lane(g, B, w.fanouts, w.dims)
    assert len(asked) == 2 and asked[1] < asked[0]
    logits = torch.full((w.num_seeds, w.classes), float("nan"), dtype=torch.float32, device="cuda")
    torch.cuda.synchronize()
    dci.dci_infer_batches([ln], g, setup["cache"], setup["seeds"], B, 3, 1, w.fanouts, w.rng_seed, 0, ws, wn, bs, logits)
    _check_lane(gu, ln, *want[3])
    _check_logits(logits[3 * B:4 * B].cpu().numpy(), oracle.sage_forward(*want[3], *(setup["tiny"][k] for k in ("w_self", "w_neigh", "bias"))))


@pytest.mark.parametrize("fused", [0, 1])
def test_void_batch_closed_beside_the_gather(setup, fused):
    """A relabel tile that gives up (forced from the host; every kernel still ends at once) voids the batch: sizes are zero, nothing is
    gathered, no logits are written, the next sync reports it once, and the lane works again."""
    dci, gu, w, g, want = (setup[k] for k in ("dci", "gu", "w", "g", "want"))
    ws, wn, bs = setup["weights"]
    ln = dci.Lane(g, B, w.fanouts, w.dims)
    ln.ctx.set_option(dci.DCI_OPT_FUSED_INPUT, fused)
    logits = torch.full((w.num_seeds, w.classes), 9.0, dtype=torch.float32, device="cuda")
    ln.x.fill_(7.0)
    torch.cuda.synchronize()
    run = lambda: dci.dci_infer_batches([ln], g, setup["cache"], setup["seeds"], B, 1, 1, w.fanouts, w.rng_seed, 0, ws, wn, bs, logits)
    ln.ctx.set_option(dci.DCI_OPT_RELABEL_SPIN_LIMIT, 200)
    ln.ctx.set_option(dci.DCI_OPT_TEST_RELABEL_FIRST_TICKET, 1)
    run()
    with pytest.raises(dci.DciError) as e:
        ln.ctx.sync()
    assert e.value.code == -3 and "relabel scan timed out" in str(e.value)
    assert ln.blocks.counts.cpu().numpy().tolist() == [0] * 17
    assert bool((ln.x == 7.0).all()) and bool((logits == 9.0).all())
    ln.ctx.set_option(dci.DCI_OPT_TEST_RELABEL_FIRST_TICKET, 0)
    ln.ctx.set_option(dci.DCI_OPT_RELABEL_SPIN_LIMIT, 1 << 24)
    run()
    gu.assert_blocks_equal(gu.blocks_to_host(ln.ctx, ln.blocks), want[1][0])
    assert bool((logits[:B] == 9.0).all()) and not bool((logits[B:2 * B] == 9.0).any())
