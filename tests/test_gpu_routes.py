"""Which kernels a forward pass takes, and that the choice changes no bits where that is promised: rows gathered first or read in
place from a cache of any alignment (DCI_OPT_FUSED_INPUT)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import paper_2503_01281_amd as dci
    from tests import gpu_util as gu
    return {"dci": dci, "gu": gu, "ctx": dci.Context(0)}


def _blocks(env, cap, fanouts, rows, num_nodes, seed):
    """Random blocks of |F_0| = rows[0], |F_1| = rows[1], ... with bounds for `cap` seeds; the batch's nodes are 0, 1, 2, ..."""
    dci = env["dci"]
    rng = np.random.default_rng(seed)
    blk = dci.Blocks(env["ctx"], num_nodes, cap, fanouts)
    blk.counts.zero_()
    blk.counts[:len(rows)] = torch.tensor(rows)
    blk.nodes.zero_()
    blk.nodes[:rows[-1]] = torch.arange(rows[-1]).cuda()
    host = []
    for h, f in enumerate(fanouts):
        deg = rng.integers(0, f + 1, rows[h])
        indptr = np.concatenate([[0], deg.cumsum()]).astype(np.int64)
        src = rng.integers(0, rows[h + 1], indptr[-1]).astype(np.int32)
        blk.blk_indptr[h][:rows[h] + 1] = torch.from_numpy(indptr).cuda()
        blk.blk_src[h][:len(src)] = torch.from_numpy(src).cuda()
        host.append((deg, src))
    return blk, host


def _weights(dims, seed):
    g = torch.Generator().manual_seed(seed)
    u = lambda *s: ((torch.rand(*s, generator=g) * 2 - 1) * (6 / sum(s)) ** 0.5).cuda()
    pairs = list(zip(dims, dims[1:]))
    return [u(*p) for p in pairs], [u(*p) for p in pairs], [u(p[1]) for p in pairs]


def _model64(model, host, x, ws, wn, bs):
    """(result, sum of magnitudes) in 64 bits"""
    v, size = x.double().cpu(), x.double().abs().cpu()
    for l, (a, c, b) in enumerate(zip(ws, wn, bs)):
        deg, src = host[len(host) - 1 - l]
        n, row = len(deg), torch.from_numpy(np.repeat(np.arange(len(deg)), deg))
        a, c, b = (t.double().cpu() for t in (a, c, b))

        def agg(t):
            s = torch.zeros(n, t.shape[1], dtype=torch.float64).index_add_(0, row, t[torch.from_numpy(src).long()])
            d = torch.from_numpy(deg)[:, None].double()
            return (s + t[:n]) / (d + 1) if model == 2 else s / d.clamp(min=1) if model == 0 else s
        y = agg(v) @ c + b
        size_y = agg(size) @ c.abs() + b.abs()
        if model != 2:
            y, size_y = y + v[:n] @ a, size_y + size[:n] @ a.abs()
        v, size = (y if l == len(ws) - 1 else y.clamp(min=0)), size_y
    return v, size


@pytest.mark.parametrize("model", [0, 1])
@pytest.mark.parametrize("F", [68, 100, 104])
def test_rows_read_in_place_from_an_unaligned_cache_give_the_same_logits(env, F, model):
    """65 to 104 columns, 256 outputs and 98,304 rows by capacity: the input layer whose kernel needs rows on 16-byte boundaries,
    before a layer whose weights are laid out as parts."""
    dci, gu, ctx = env["dci"], env["gu"], env["ctx"]
    n, dims = 5000, (F, 256, 64)
    feat = torch.randn(n, F, generator=torch.Generator().manual_seed(F))
    g = dci.Graph(torch.zeros(n + 1, dtype=torch.int64).cuda(), torch.zeros(1, dtype=torch.int64).cuda(), feat.cuda())
    blk, host = _blocks(env, 20_000, (4, 5), (700, 2100, 4700), 10**7, F)
    assert blk.cap_nodes[1] >= 98304
    ws, wn, bs = _weights(dims, F + model)
    rows = torch.randperm(n, generator=torch.Generator().manual_seed(2))[:n // 2]
    remap = torch.full((n,), -1, dtype=torch.int32)
    remap[rows] = torch.arange(len(rows), dtype=torch.int32)
    empty = torch.zeros(0, dtype=torch.int64).cuda()
    out = []
    for shift in (0, 1, 2):
        buf = torch.empty(len(rows) * F + 4, dtype=torch.float32, device="cuda")
        rows_at = buf[shift:shift + len(rows) * F].view(-1, F)
        rows_at.copy_(feat[rows])
        assert rows_at.data_ptr() % 16 == 4 * shift
        cache = dci.Cache.from_arrays(torch.full((n,), -1, dtype=torch.int32).cuda(), torch.zeros(1, dtype=torch.int64).cuda(), empty,
                                      remap.cuda(), rows_at)
        for fused in (0, 1):
            x = torch.zeros(blk.cap_nodes[-1], F, dtype=torch.float32, device="cuda")
            y = torch.full((blk.cap_nodes[0], dims[-1]), float("nan"), dtype=torch.float32, device="cuda")
            if fused:
                dci.dci_gather_forward(ctx, g, cache, blk, x, model, ws, wn, bs, y)
            else:
                dci.dci_gather_features(ctx, g, cache, blk.nodes, blk.cap_nodes[-1], x, n_dev=blk.n_input_dev())
                dci.dci_gnn_forward(ctx, blk, x, model, ws, wn, bs, y)
            ctx.sync()
            out.append(y[:700].cpu())
    want, size = _model64(model, host, feat[:4700], ws, wn, bs)
    assert bool(((out[0].double() - want).abs() <= size * 2.0 ** -24 * (sum(dims) + 30)).all())
    for o in out[1:]:
        assert o.numpy().tobytes() == out[0].numpy().tobytes()


def _one_layer(env, M, cap, fan, D, N, model, seed, deg=None):
    """One layer through dci_gather_forward on gathered rows: (result, 64-bit result, sum of magnitudes, launches per kernel class)"""
    dci, ctx = env["dci"], env["ctx"]
    n_in = M + 7
    blk, host = _blocks(env, cap, (min(fan, 64),), (M, n_in), 10**7, seed)
    if deg is not None:
        src = np.random.default_rng(seed).integers(0, n_in, deg.sum()).astype(np.int32)
        blk.blk_indptr[0][:M + 1] = torch.from_numpy(np.concatenate([[0], deg.cumsum()])).cuda()
        blk.blk_src[0][:len(src)] = torch.from_numpy(src).cuda()
        host = [(deg, src)]
    feat = torch.randn(n_in, D, generator=torch.Generator().manual_seed(seed))
    g = dci.Graph(torch.zeros(n_in + 1, dtype=torch.int64).cuda(), torch.zeros(1, dtype=torch.int64).cuda(), feat.cuda())
    ws, wn, bs = _weights((D, N), seed + 1)
    x = torch.zeros(blk.cap_nodes[-1], D, dtype=torch.float32, device="cuda")
    y = torch.full((blk.cap_nodes[0], N), float("nan"), dtype=torch.float32, device="cuda")
    ctx.timing_enable(dci.KERNEL_CLASSES)
    dci.dci_gather_forward(ctx, g, None, blk, x, model, None if model == 2 else ws, wn, bs, y)
    n = {k: v[1] for k, v in ctx.timing_read().items()}
    ctx.timing_enable([])
    assert bool(torch.isnan(y[M:]).all()), "rows beyond the batch were written"
    want, size = _model64(model, host, feat, ws, wn, bs)
    return y[:M].cpu(), want, size, n


@pytest.mark.parametrize("model", [0, 1, 2])
@pytest.mark.parametrize("M,cap,D,N", [(70, 40000, 128, 64), (70, 40000, 160, 200), (70, 20000, 96, 100)])
def test_lists_as_long_as_the_places_for_their_sources(env, model, M, cap, D, N):
    """Rows with 0, 1, 31 to 33, 63 to 65 and 100 sources, next to each other, in tiles of many rows."""
    deg = np.random.default_rng(D).choice([0, 1, 8, 9, 31, 32, 33, 40, 63, 64, 65, 100], M)
    deg[:3] = (64, 65, 0)
    got, want, size, n = _one_layer(env, M, cap, 64, D, N, model, D + N, deg)
    assert n["mean_in"] == 0 and n["linear_in"] == 1        # one kernel
    assert bool(((got.double() - want).abs() <= size * 2.0 ** -24 * (100 + D / 4 + 8)).all())
