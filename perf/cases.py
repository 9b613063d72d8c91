"""The work that is timed on this framework: what its users have it do, as plain cases.

Three kinds of work, each through the public calls of ``paper_2503_01281_amd``:

  infer  mini-batches through sampling, feature loading and the model (``dci_infer_batches``): one batch on the
         caller's own stream (a request that is answered at once) or several batches over one or more lanes (a
         pass over a test set).  ``fused`` is DCI_OPT_FUSED_INPUT: 1 reads cached neighbour rows in place, 0 (the
         option's default) gathers every input row first.
  load   a mini-batch and its feature rows for a model that lives elsewhere: ``dci_sample_khop`` and
         ``dci_gather_features`` with statistics, then a wait, because that model needs the batch's sizes.
  prep   what precedes inference: the access counters of eight pre-sampled batches (``dci_presample_count``, features
         loaded as well, as Eq. (1) wants it) and the two caches filled from them (``dci_fill_caches``).

Graphs are R-MAT graphs with random labels, as in ``synth``, but drawn on the GPU from the case's seed; features are
N(0, 1), weights Glorot-uniform, seed nodes distinct and uniform.  ``host`` puts the graph and the features into pinned
host memory, which a cache miss reads over the host link; where everything is cached nothing of them is read during
inference, and they stay on the GPU, which is quicker to make.  ``host_bounds`` puts only the list bounds there, as for
graphs whose neighbour ids do not fit into pinned memory.  ``cached`` is the cache budget as a share of the graph's and
the features' bytes together (1: all of it).
"""
import math

import torch

import paper_2503_01281_amd as dci

A, B, C = 0.57, 0.19, 0.19  # R-MAT quadrants
LOW = A + B                 # probability of a zero bit in a label, for sources and destinations alike
N_PRESAMPLE = 8
RNG_PRESAMPLE = 1 << 31     # RNG batch indices of the pre-sampled batches
T_SAMPLE, T_FEATURE = 1, 9  # stage times for Eq. (1), fixed so that the caches depend on the inputs alone (the largest
                            # configuration measures about this ratio)


def _case(name, kind, nodes, edges, feat, fanouts, batch, **kw):
    c = dict(name=name, kind=kind, nodes=nodes, edges=edges, feat=feat, fanouts=fanouts, batch=batch, batches=1, lanes=1,
             hidden=256, classes=47, model=0, fused=1, cached=1.0, host=0, host_bounds=0, topk=0)
    c.update(kw)
    return c


def listed():
    return [
        # a request of a few seed nodes against the Ogbn-products-shaped graph: latency is all that counts
        _case("request 16 seeds", "infer", 2_449_029, 61_900_000, 100, "5,10,15", 16),
        # the smallest configuration, its caches a fifth of the data, misses over the host link
        _case("tiny, part cached", "infer", 16_384, 163_840, 64, "5,10", 256, hidden=64, classes=16, cached=0.2, host=1),
        # a Reddit-shaped batch: wide rows, everything cached
        _case("medium batch", "infer", 232_965, 114_600_000, 602, "5,10,15", 1024, classes=41),
        # test-set pass, four batches in flight
        _case("large pass, 4 lanes", "infer", 2_449_029, 61_900_000, 100, "5,10,15", 4096, batches=8, lanes=4),
        # test-set pass with a graph many times the size of the on-chip caches (a quarter of the largest configuration's nodes,
        # so that it can be made in a second), list bounds of the nodes outside the adjacency cache over the host link
        _case("huge pass", "infer", 24_000_000, 350_000_000, 128, "5,10,15", 4096, batches=8, classes=172, cached=0.93,
              host_bounds=1),
        # two hops with a wide second fan-out, wide rows, large batches, the option's default route (gather, then model)
        _case("social, two hops", "infer", 4_000_000, 110_000_000, 256, "10,25", 8192, classes=64, fused=0),
        # the other models of the paper's Table III on its other datasets' shapes
        _case("yelp, sum", "infer", 716_480, 6_977_410, 300, "5,10,15", 4096, hidden=128, classes=100, model=1),
        _case("amazon, gcn", "infer", 1_598_960, 66_000_000, 200, "5,10,15", 4096, hidden=128, classes=107, model=2, fused=0),
        # nothing divides anything: odd widths, odd batches
        _case("odd widths", "infer", 300_007, 3_000_001, 75, "2,4,8", 1001, batches=3, hidden=130, classes=41),
        # the host link: a fifth of the data cached, batches for a model elsewhere
        _case("loader, part cached", "load", 1_200_011, 30_000_000, 100, "5,10,15", 2048, cached=0.2, host=1),
        # preparation from host memory with the paper's feature rule, and on the GPU with the feature order by count
        _case("preparation, host", "prep", 1_200_011, 30_000_000, 100, "5,10,15", 2048, cached=0.5, host=1),
        _case("preparation, top-k", "prep", 2_449_029, 61_900_000, 100, "2,4,8", 4096, cached=0.3, topk=1),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["infer"] * 4 + ["load", "prep"])
    cached = rng.choice([1.0, 1.0, rng.uniform(0.1, 0.9)])
    host = 1 if cached < 1.0 and rng.random() < 0.7 else 0
    nodes = log_int(12_000, 2_400_000)
    edges = min(int(nodes * math.exp(rng.uniform(math.log(7), math.log(300)))), 60_000_000)
    feat = log_int(33, 620)
    if rng.random() < 0.6:
        feat = max(32, feat // 4 * 4)
    if host or kind == "prep":  # bytes to be pinned, or to be copied by every fill
        nodes = max(12_000, min(nodes, 400_000_000 // (4 * feat)))
        edges = min(edges, 25_000_000)
    batch = log_int(16, 6000)
    batches = 1 if rng.random() < 0.5 else rng.randint(2, 6)
    batches = max(1, min(batches, (6000 if host else 16_000) // batch, nodes // (2 * batch)))
    batch = min(batch, nodes // 8)
    return dict(kind=kind, nodes=nodes, edges=edges, feat=feat,
                fanouts=rng.choice(["5,10,15", "5,10,15", "2,4,8", "2,2,2", "5,10", "10,25"]), batch=batch,
                batches=batches if kind == "infer" else 1, lanes=rng.choice([1, 4]) if batches > 1 and kind == "infer" else 1,
                hidden=rng.choice([64, 128, 256, 256, rng.randint(40, 260)]), classes=rng.randint(7, 172),
                model=rng.choice([0, 0, 1, 2]), fused=rng.choice([0, 1]), cached=round(cached, 3), host=host, host_bounds=0,
                topk=rng.choice([0, 1]))


# ---- inputs --------------------------------------------------------------------------------------


def _fanouts(case):
    return tuple(int(f) for f in case["fanouts"].split(","))


def _dims(case):
    return (case["feat"],) + (case["hidden"],) * (len(_fanouts(case)) - 1) + (case["classes"],)


def _scale(case):
    return max(1, math.ceil(math.log2(case["nodes"])))


def _rmat(case, gen):
    """(indptr, indices) on the GPU: R-MAT labels of `scale` bits, scaled down to the node count and shuffled."""
    n, e, s = case["nodes"], case["edges"], _scale(case)
    perm = torch.randperm(n, generator=gen, device="cuda")
    keys = torch.empty(e, dtype=torch.int64, device="cuda")
    step = 1 << 25
    for lo in range(0, e, step):
        m = min(step, e - lo)
        src = torch.zeros(m, dtype=torch.int32, device="cuda")
        dst = torch.zeros(m, dtype=torch.int32, device="cuda")
        for _ in range(s):
            u = torch.rand(m, generator=gen, device="cuda")
            d_bit = u >= LOW
            src.mul_(2).add_((u >= A) & ~d_bit | (u >= A + B + C))
            dst.mul_(2).add_(d_bit)
        keys[lo:lo + m] = perm[(dst.long() * n) >> s] * n + perm[(src.long() * n) >> s]
    keys = keys.sort()[0]
    dst = torch.div(keys, n, rounding_mode="floor")
    indptr = torch.searchsorted(dst, torch.arange(n + 1, device="cuda"))
    del dst
    return indptr, keys.remainder_(n)


def _to_host(t):
    h = dci.pinned_empty(t.numel(), t.dtype).view(t.shape)
    h.copy_(t)
    return h


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    n, f, fanouts, dims = case["nodes"], case["feat"], _fanouts(case), _dims(case)
    indptr, indices = _rmat(case, gen)
    feat = torch.randn(n, f, generator=gen, device="cuda")
    n_seeds = case["batch"] * case["batches"] - (case["batch"] // 3 if case["batches"] > 1 else 0)  # the last batch of a pass is short
    seeds = torch.randperm(n, generator=gen, device="cuda")[:n_seeds].contiguous()
    pre_seeds = torch.randperm(n, generator=gen, device="cuda")[:case["batch"] * N_PRESAMPLE].contiguous()
    if case["host"] or case["host_bounds"]:
        indptr = _to_host(indptr)
    if case["host"]:
        indices, feat = _to_host(indices), _to_host(feat)
    g = dci.Graph(indptr, indices, feat)
    s = dict(case=case, seed=seed, graph=g, seeds=seeds, fanouts=fanouts,
             budget=int(case["cached"] * (8 * (n + 1 + case["edges"]) + 4 * n * f)))
    stream = torch.cuda.current_stream()
    if case["kind"] == "prep":
        s.update(seeds=pre_seeds, ctx=dci.Context(0, stream=stream))
        s["x"] = torch.empty(dci.blocks_bounds(n, case["batch"], fanouts)[0][-1], f, device="cuda")
        s["counts"] = [torch.zeros(n, dtype=torch.int32, device="cuda") for _ in range(2)]
        s["stats"] = torch.zeros(dci.STATS_WORDS, dtype=torch.int64, device="cuda")
        s["lists"] = torch.zeros(min(s["budget"] // 8, n + 1 + case["edges"]), dtype=torch.int64, device="cuda")
        torch.cuda.synchronize()
        return s
    # the caches that the program filled before: counters of eight batches, then the fill
    lanes = [dci.Lane(g, case["batch"], fanouts, dims, stream=stream if k == 0 else None) for k in range(case["lanes"])]
    counts = [torch.zeros(n, dtype=torch.int32, device="cuda") for _ in range(2)]
    ctx = lanes[0].ctx
    dci.dci_presample_count(ctx, g, None, pre_seeds, case["batch"], 0, N_PRESAMPLE, RNG_PRESAMPLE, fanouts, seed, *counts)
    s["cache"] = dci.dci_fill_caches(ctx, g, *counts, s["budget"], T_SAMPLE, T_FEATURE, case["topk"])
    s["lanes"] = lanes
    for ln in lanes:
        for t in [ln.x, ln.blocks.nodes] + ln.blocks.blk_indptr + ln.blocks.blk_src:
            t.zero_()
    if case["kind"] == "load":
        s["stats"] = torch.zeros(dci.STATS_WORDS, dtype=torch.int64, device="cuda")
    else:
        for ln in lanes:
            ln.ctx.set_option(dci.DCI_OPT_FUSED_INPUT, case["fused"])

        def uniform(*shape):
            bound = math.sqrt(6.0 / sum(shape)) if len(shape) == 2 else 0.1
            return (torch.rand(*shape, generator=gen, device="cuda") * 2 - 1) * bound

        pairs = list(zip(dims, dims[1:]))
        s["w_self"] = None if case["model"] == dci.DCI_MODEL_GCN_AVG else [uniform(*p) for p in pairs]
        s["w_neigh"] = [uniform(*p) for p in pairs]
        s["bias"] = [uniform(p[1]) for p in pairs]
        s["logits"] = torch.empty(seeds.numel(), dims[-1], device="cuda")
    torch.cuda.synchronize()
    return s


# ---- one pass ------------------------------------------------------------------------------------


def run(s):
    return {"infer": _infer, "load": _load, "prep": _prep}[s["case"]["kind"]](s)


def _infer(s):
    c = s["case"]
    dci.dci_infer_batches(s["lanes"], s["graph"], s["cache"], s["seeds"], c["batch"], 0, c["batches"], s["fanouts"], s["seed"],
                          c["model"], s["w_self"], s["w_neigh"], s["bias"], s["logits"])
    if len(s["lanes"]) > 1:  # the lanes have streams of their own: wait for them before the logits are read
        for ln in s["lanes"]:
            ln.ctx.sync()
    return dict(logits=s["logits"], lanes=[_blocks(ln.blocks) for ln in s["lanes"]],
                x=None if c["fused"] else [ln.x for ln in s["lanes"]])


def _blocks(blk):
    """The batch that a lane holds, in the buffers it lives in (made of zeros by prepare, so that what a batch leaves
    unused is the same for everybody)."""
    return dict(nodes=blk.nodes, indptr=blk.blk_indptr, src=blk.blk_src, counts=blk.counts)


def _load(s):
    ln, g, stats = s["lanes"][0], s["graph"], s["stats"]
    ctx, blk = ln.ctx, ln.blocks
    stats.zero_()
    dci.dci_sample_khop(ctx, g, s["cache"], s["seeds"], 0, s["fanouts"], s["seed"], blk, stats)
    dci.dci_gather_features(ctx, g, s["cache"], blk.nodes, blk.cap_nodes[-1], ln.x, n_dev=blk.n_input_dev(), stats=stats)
    ctx.sync()  # the other model wants the batch's sizes on the host
    return dict(_blocks(blk), x=ln.x, stats=stats)


def _prep(s):
    c, g, ctx, stats = s["case"], s["graph"], s["ctx"], s["stats"]
    feat_count, adj_count = s["counts"]
    for t in (feat_count, adj_count, stats):
        t.zero_()
    dci.dci_presample_count(ctx, g, None, s["seeds"], c["batch"], 0, N_PRESAMPLE, RNG_PRESAMPLE, s["fanouts"], s["seed"],
                            feat_count, adj_count, feat_scratch=s["x"], stats=stats)
    cache = dci.dci_fill_caches(ctx, g, feat_count, adj_count, s["budget"], T_SAMPLE, T_FEATURE, c["topk"])
    buf = cache.buf[cache.buf_offset:]
    # how much of its share the adjacency cache fills differs from graph to graph: kept in a buffer of one size
    adj_at, adj_len = (cache.feat_bytes + 7) // 8 * 8, cache.adj_bytes if cache.adj_nodes else 0
    s["lists"][:adj_len // 8].copy_(buf[adj_at:adj_at + adj_len].view(torch.int64))
    return dict(feat_count=feat_count, adj_count=adj_count, sampled=stats[:8], adj_remap=cache.adj_remap, feat_remap=cache.feat_remap,
                rows=buf[:cache.feat_bytes].view(torch.float32), lists=s["lists"])


# ---- what a pass cannot do without -----------------------------------------------------------------


def _batch_sizes(case):
    """Expected |F_h| (h = 0..L) and edges per hop of one batch: nodes fall into classes by the number of one-bits of
    their R-MAT label; within a class all are alike, and a hop reaches a node with a probability that follows from the
    number of edges and the class's share of the sources."""
    n, e, s = case["nodes"], case["edges"], _scale(case)
    size = [math.comb(s, k) * n / 2.0 ** s for k in range(s + 1)]
    share = [LOW ** (s - k) * (1 - LOW) ** k * 2.0 ** s / n for k in range(s + 1)]  # of all edges, per node of the class
    q = [min(1.0, case["batch"] / n)] * (s + 1)
    nodes, edges = [case["batch"]], []
    for f in _fanouts(case):
        e_h = sum(c * p * min(f, e * w) for c, p, w in zip(size, q, share))
        q = [1 - (1 - p) * math.exp(-min(700.0, e_h * w)) for p, w in zip(q, share)]
        edges.append(e_h)
        nodes.append(sum(c * p for c, p in zip(size, q)))
    return nodes, edges


def work(case):
    nodes, edges = _batch_sizes(case)
    dims, layers = _dims(case), len(edges)
    # sampling: a frontier node's two list bounds, the neighbour ids of the edges taken; the batch it leaves: node ids, row
    # offsets, local ids
    sample = 16 * nodes[-2] + 8 * sum(edges) + 8 * nodes[-1] + 8 * sum(nodes[:-1]) + 4 * sum(edges)
    rows = 4 * case["feat"] * nodes[-1]
    if case["kind"] == "load":
        return {"bytes": sample + 2 * rows, "flops": 0.0}
    if case["kind"] == "prep":
        total = 8 * (case["nodes"] + 1 + case["edges"]) + 4 * case["nodes"] * case["feat"]
        fill = 2 * case["cached"] * total + 4 * 4 * case["nodes"] + 8 * case["nodes"]  # copies, counters and remaps, degrees
        return {"bytes": N_PRESAMPLE * (sample + 2 * rows) + fill, "flops": 0.0}
    ops = 1 if case["model"] == 2 else 2
    flops = sum(2.0 * nodes[layers - 1 - l] * ops * dims[l] * dims[l + 1] + dims[l] * edges[layers - 1 - l] for l in range(layers))
    weights = 4 * sum(ops * i * o + o for i, o in zip(dims, dims[1:]))
    return {"bytes": case["batches"] * (sample + rows + 4 * case["batch"] * dims[-1]) + weights, "flops": case["batches"] * flops}


def tolerance(case):
    # sampled batches, copied rows, counters and caches are defined to the bit; logits are sums of up to a thousand or so
    # 32-bit products, three layers deep
    return {"rel": 1e-5} if case["kind"] == "infer" else "exact"
