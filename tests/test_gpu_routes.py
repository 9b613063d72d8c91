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


def _forward(env, cap, fanouts, rows, dims, model, seed, deg=None, shift=0):
    """dci_gather_forward on gathered rows: (result, 64-bit result, sum of magnitudes, launches per kernel class).  deg: list
    lengths of the input layer's block; shift: numbers that x begins beyond a 16-byte boundary."""
    dci, ctx = env["dci"], env["ctx"]
    blk, host = _blocks(env, cap, fanouts, rows, 10**7, seed)
    if deg is not None:
        h = len(fanouts) - 1
        src = np.random.default_rng(seed).integers(0, rows[-1], deg.sum()).astype(np.int32)
        blk.blk_indptr[h][:rows[h] + 1] = torch.from_numpy(np.concatenate([[0], deg.cumsum()])).cuda()
        blk.blk_src[h][:len(src)] = torch.from_numpy(src).cuda()
        host[h] = (deg, src)
    n = rows[-1]
    feat = torch.randn(n, dims[0], generator=torch.Generator().manual_seed(seed))
    g = dci.Graph(torch.zeros(n + 1, dtype=torch.int64).cuda(), torch.zeros(1, dtype=torch.int64).cuda(), feat.cuda())
    ws, wn, bs = _weights(dims, seed + 1)
    x = torch.zeros(blk.cap_nodes[-1] * dims[0] + shift, dtype=torch.float32, device="cuda")[shift:].view(-1, dims[0])
    y = torch.full((blk.cap_nodes[0], dims[-1]), float("nan"), dtype=torch.float32, device="cuda")
    ctx.timing_enable(dci.KERNEL_CLASSES)
    dci.dci_gather_forward(ctx, g, None, blk, x, model, None if model == 2 else ws, wn, bs, y)
    launches = {k: v[1] for k, v in ctx.timing_read().items()}
    ctx.timing_enable([])
    assert bool(torch.isnan(y[rows[0]:]).all()), "rows beyond the batch were written"
    want, size = _model64(model, host, feat, ws, wn, bs)
    return y[:rows[0]].cpu().double(), want, size, launches


def _close(got, want, size, fanouts, dims):
    # a mean of f rows is off by f 2^-24 of their magnitudes, a contraction of 2 D products by less than D / 4, layer after layer
    return bool(((got - want).abs() <= size * 2.0 ** -24 * (sum(fanouts) + sum(dims) / 4 + 8)).all())


@pytest.mark.parametrize("model", [0, 1, 2])
@pytest.mark.parametrize("M,cap,D,N", [(70, 40000, 128, 64), (70, 40000, 160, 200), (70, 20000, 96, 100)])
def test_lists_as_long_as_the_places_for_their_sources(env, model, M, cap, D, N):
    """Rows with 0, 1, 31 to 33, 63 to 65 and 100 sources, next to each other, in tiles of many rows."""
    deg = np.random.default_rng(D).choice([0, 1, 8, 9, 31, 32, 33, 40, 63, 64, 65, 100], M)
    deg[:3] = (64, 65, 0)
    got, want, size, n = _forward(env, cap, (64,), (M, M + 7), (D, N), model, D + N, deg)
    assert n["mean_in"] == 0 and n["linear_in"] == 1        # one kernel
    assert _close(got, want, size, (100,), (D, N))


@pytest.mark.parametrize("model", [0, 1, 2])
@pytest.mark.parametrize("D", [100, 260])
def test_lists_of_few_rows_that_are_longer_than_most(env, model, D):
    """Rows with more sources than the block has room for on average, in a layer of few rows."""
    deg = np.array([100, 0, 65, 64, 63, 1, 0, 8, 9, 66, 0, 2, 7, 0, 0, 15, 16, 17, 0, 40])
    got, want, size, n = _forward(env, 64, (10,), (20, 27), (D, 70), model, D, deg)
    assert n["mean_in"] == 0 and n["linear_in"] == 1
    assert _close(got, want, size, (100,), (D, 70))


@pytest.mark.parametrize("cap,fan,D,N,kernels", [
    # a workgroup of 16 rows by 64 columns for every compute unit, and one more; short and long lists there
    (4096, 5, 256, 64, 1), (4112, 5, 256, 64, 1), (4112, 64, 100, 64, 1), (4112, 41, 256, 128, 2), (1024, 39, 256, 256, 1), (1024, 40, 256, 256, 2),
    (1024, 38, 260, 200, 1), (1024, 39, 260, 200, 2), (1024, 16, 602, 41, 1), (1024, 17, 602, 41, 1),
    (1024, 21, 602, 41, 1), (1024, 22, 602, 41, 2), (1040, 64, 256, 100, 2), (1024, 64, 256, 100, 1)])
def test_kernels_of_a_layer_of_few_rows(env, cap, fan, D, N, kernels):
    got, want, size, n = _forward(env, cap, (fan,), (cap, cap + 100), (D, N), 0, cap + D + N)
    assert n["mean_in"] + n["linear_in"] == kernels
    assert _close(got, want, size, (fan,), (D, N))


@pytest.mark.parametrize("cap,fan,D,N,kernels", [
    # few tiles, by an estimate of the rows (a fifth of the bound, 4 cap): 16, 32 and 64 columns to a wavefront, one column group and
    # several
    (2000, 7, 96, 192, 1), (2000, 7, 33, 256, 1), (1500, 5, 68, 300, 1), (2000, 5, 40, 300, 1), (2000, 5, 64, 512, 1),
    (4000, 9, 31, 257, 1), (8000, 9, 36, 193, 1),
    # more tiles than that
    (14_000, 6, 48, 64, 1), (14_000, 6, 48, 65, 1), (14_000, 6, 48, 129, 1), (14_000, 2, 64, 257, 2), (14_000, 2, 64, 384, 2),
    (14_000, 2, 64, 385, 1), (14_000, 5, 31, 1030, 1),
    # lists as long as they may be, and longer
    (2000, 39, 256, 192, 1), (2000, 40, 256, 192, 2), (2000, 33, 300, 256, 1), (2000, 34, 300, 256, 2),
    (14_000, 20, 100, 256, 1), (14_000, 21, 100, 256, 2), (14_000, 15, 100, 1024, 1), (14_000, 16, 100, 1024, 2),
    (14_000, 64, 128, 256, 1), (14_000, 42, 128, 512, 1), (14_000, 43, 128, 512, 2), (14_000, 25, 300, 256, 2)])
def test_kernels_of_an_input_layer(env, cap, fan, D, N, kernels):
    fanouts, dims = (1, 1, fan), (D, N, 8, 5)
    got, want, size, n = _forward(env, cap, fanouts, (100, 170, 300, 1000), dims, 0, cap + D + N)
    assert n["mean_in"] + n["linear_in"] == kernels
    assert _close(got, want, size, fanouts, dims)


@pytest.mark.parametrize("model", [0, 1])
@pytest.mark.parametrize("fan,D,N,tiles", [
    (10, 100, 256, 0), (11, 68, 256, 0), (16, 100, 256, 0), (15, 104, 256, 0), (16, 128, 512, 0),
    # rows that are no whole 128-byte lines: the lists' length times the column groups up to 60; those that are: times one more, up to 128
    (15, 112, 1024, 0), (16, 112, 1024, 1), (12, 112, 1280, 0), (13, 112, 1280, 1), (16, 128, 1024, 0), (14, 128, 2048, 0), (15, 128, 2048, 1)])
def test_input_layers_of_many_rows_with_11_to_16_sources(env, model, fan, D, N, tiles):
    """At least 98,304 rows by capacity, inputs of up to 128 columns: one kernel, with three-part products, or with fp32 instructions
    (tiles) where that one would put the rows together too often.  The latter needs rows on 16-byte boundaries: elsewhere the layer is two
    kernels."""
    fanouts, dims = (1, 1, fan), (D, N, 8, 5)
    for shift in (0, 1):
        got, want, size, n = _forward(env, 25_000, fanouts, (100, 170, 3001, 4000), dims, model, D + N + fan, shift=shift)
        assert n["mean_in"] + n["linear_in"] == (2 if tiles and shift else 1)
        assert _close(got, want, size, fanouts, dims)


@pytest.mark.parametrize("cap,kernels", [(8000, 1), (5000, 2)])
def test_parts_fit_where_the_aggregated_rows_would_be_or_not(env, cap, kernels):
    """98,304 bytes of parts of 2 x 4 x 256 weights, 16 bytes to a row."""
    got, want, size, n = _forward(env, cap, (3,), (3000, 3007), (4, 256), 0, cap)
    assert n["mean_in"] + n["linear_in"] == kernels
    assert _close(got, want, size, (3,), (4, 256))


@pytest.mark.parametrize("cap,N,kernels", [
    # parts of 2 x 6 x 192 weights for 130 and 192 outputs (73,728 bytes) and of 2 x 6 x 320 for 300, 24 bytes to a row; too little for all the
    # columns that the wavefronts of a column group could have (256, 256, 512)
    (3400, 130, 1), (2400, 130, 2), (3400, 192, 1), (2900, 192, 2), (5120, 300, 1), (4900, 300, 2)])
def test_parts_take_whole_blocks_of_64_columns_and_no_more(env, cap, N, kernels):
    got, want, size, n = _forward(env, cap, (3,), (cap - 100, cap), (6, N), 0, cap + N)
    assert n["mean_in"] + n["linear_in"] == kernels
    assert _close(got, want, size, (3,), (6, N))


@pytest.mark.parametrize("model", [0, 2])
@pytest.mark.parametrize("N,cap,rows", [(64, 10_000, 20_011), (100, 10_000, 20_011), (600, 10_000, 20_011),   # 16, 32, 64 columns
                                        (256, 2000, 8000), (500, 2000, 8000)])                             # 16, 32
def test_more_tiles_than_workgroups_in_several_column_groups(env, model, N, cap, rows):
    """Several tiles to a workgroup: the next tile's weights are asked for while the last one is multiplied, and they are another
    column group's."""
    fanouts, dims = (1, 1, 3), (36, N, 8, 5)
    got, want, size, n = _forward(env, cap, fanouts, (100, 170, rows, rows + 7), dims, model, N)
    assert n["mean_in"] == 0
    assert _close(got, want, size, fanouts, dims)


def test_more_tiles_than_flags(env):
    """More than 64 tiles to a workgroup: tiles share the flag that has one made again, and are made again with it."""
    dci, ctx = env["dci"], env["ctx"]
    M, D, N = 1_300_003, 4, 64
    blk = dci.Blocks(ctx, 10**7, M, (1,))
    blk.counts.zero_()
    blk.counts[0] = blk.counts[1] = M
    blk.blk_indptr[0][:M + 1] = torch.arange(M + 1).cuda()
    src = torch.randperm(M, generator=torch.Generator().manual_seed(3))
    blk.blk_src[0][:M] = src.int().cuda()
    x = torch.randn(M, D, generator=torch.Generator().manual_seed(4))
    x[7, 1], x[M - 5, 2] = float("inf"), 1e33
    x_dev = torch.zeros(blk.cap_nodes[1], D, dtype=torch.float32, device="cuda")
    x_dev[:M] = x.cuda()
    ws, wn, bs = _weights((D, N), 5)
    y = torch.empty(blk.cap_nodes[0], N, dtype=torch.float32, device="cuda")
    dci.dci_gnn_forward(ctx, blk, x_dev, 0, ws, wn, bs, y)
    ctx.sync()
    a, c, b = (t[0].double().cpu() for t in (ws, wn, bs))
    xd = x.double()
    want = xd @ a + xd[src] @ c + b
    size = xd.abs() @ a.abs() + xd.abs()[src] @ c.abs() + b.abs()
    got = y[:M].cpu().double()
    fin = torch.isfinite(want)
    assert int((~fin).sum()) == 2 * N and bool((got[~fin] == want[~fin]).all())
    assert bool(((got - want).abs()[fin] <= (size * 2.0 ** -24 * 12)[fin]).all())


def test_parts_are_laid_out_again_after_a_layer_that_takes_their_place(env):
    """Three layers: one kernel, aggregation and dense layer apart (its aggregated rows go where the parts of the weights were), one
    kernel.  Gathered rows and rows read in place give the same logits."""
    dci, ctx = env["dci"], env["ctx"]
    dims, fanouts, rows = (64, 100, 128, 65), (2, 40, 2), (500, 1400, 5000, 9000)
    n = rows[-1]
    feat = torch.randn(n, dims[0], generator=torch.Generator().manual_seed(1))
    g = dci.Graph(torch.zeros(n + 1, dtype=torch.int64).cuda(), torch.zeros(1, dtype=torch.int64).cuda(), feat.cuda())
    blk, host = _blocks(env, 12_000, fanouts, rows, 10**7, 6)
    ws, wn, bs = _weights(dims, 7)
    remap = torch.arange(n, dtype=torch.int32)
    cache = dci.Cache.from_arrays(torch.full((n,), -1, dtype=torch.int32).cuda(), torch.zeros(1, dtype=torch.int64).cuda(),
                                  torch.zeros(0, dtype=torch.int64).cuda(), remap.cuda(), feat.cuda())
    x = torch.zeros(blk.cap_nodes[-1], dims[0], dtype=torch.float32, device="cuda")
    y = [torch.full((blk.cap_nodes[0], dims[-1]), float("nan"), dtype=torch.float32, device="cuda") for _ in range(2)]
    ctx.timing_enable(dci.KERNEL_CLASSES)
    dci.dci_gather_forward(ctx, g, cache, blk, x, 0, ws, wn, bs, y[0])
    launches = {k: v[1] for k, v in ctx.timing_read().items()}
    ctx.timing_enable([])
    assert launches["mean_in"] == 0 and launches["mean"] == 1 and launches["linear"] == 2
    dci.dci_gather_features(ctx, g, cache, blk.nodes, blk.cap_nodes[-1], x, n_dev=blk.n_input_dev())
    dci.dci_gnn_forward(ctx, blk, x, 0, ws, wn, bs, y[1])
    ctx.sync()
    want, size = _model64(0, host, feat, ws, wn, bs)
    assert bool(((y[0][:500].double().cpu() - want).abs() <= size * 2.0 ** -24 * (sum(dims) + sum(fanouts))).all())
    assert y[0][:500].cpu().numpy().tobytes() == y[1][:500].cpu().numpy().tobytes()
