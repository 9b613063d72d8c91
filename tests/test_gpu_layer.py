"""A layer as one kernel (dci_layer.hip) at the edges of its tiles: rows around 16 and 32, input widths around the steps of
32, 64 and 256 columns and ragged, output widths around 16 C x 4, row lists shorter and longer than what LDS keeps, the
three models; and what its three-part products cannot hold (infinities, NaN, the largest and the smallest numbers).

The bound on a result: a mean of up to f rows is off by (f + 1) 2^-24 of the sum of their magnitudes, a contraction of K products
added up one after the other by K 2^-24 of the sum of theirs; the kernels add 16 at a time or more, so K / 8 is ample."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import paper_2503_01281_amd as dci
    from tests import gpu_util as gu
    return {"dci": dci, "gu": gu, "ctx": dci.Context(0)}


def _run(env, M, D, N, fan, model, cap, seed, poke=None, scale=1.0):
    dci, gu, ctx = env["dci"], env["gu"], env["ctx"]
    rng = np.random.default_rng(seed)
    n_src = M + 5
    blk = dci.Blocks(ctx, 10**7, cap, (min(fan, 64),))
    deg = rng.integers(0, fan + 1, M)
    deg[rng.integers(0, M)] = fan
    while deg.sum() > blk.cap_edges[0]:
        deg //= 2
    indptr = np.concatenate([[0], deg.cumsum()]).astype(np.int64)
    src = rng.integers(0, n_src, indptr[-1]).astype(np.int32)
    blk.counts.zero_()
    blk.counts[0], blk.counts[1] = M, n_src
    blk.blk_indptr[0][:M + 1] = torch.from_numpy(indptr).cuda()
    if len(src):
        blk.blk_src[0][:len(src)] = torch.from_numpy(src).cuda()
    x = (rng.standard_normal((n_src, D)) * scale).astype(np.float32)
    ws, wn = (rng.uniform(-1, 1, (2, D, N)) * np.sqrt(6 / (D + N))).astype(np.float32)
    b = (rng.uniform(-0.1, 0.1, N) * scale).astype(np.float32)
    if poke:
        poke(x, ws, wn)
    x_dev = torch.zeros(max(n_src, blk.cap_nodes[0]), D, dtype=torch.float32, device="cuda")
    x_dev[:n_src] = torch.from_numpy(x).cuda()
    out = torch.full((blk.cap_nodes[0], N), float("nan"), dtype=torch.float32, device="cuda")
    ctx.timing_enable(["mean_in"])
    dci.dci_gnn_forward(ctx, blk, x_dev, model, None if model == 2 else [gu.dev(ws)], [gu.dev(wn)], [gu.dev(b)], out)
    env["one kernel"] = ctx.timing_read()["mean_in"][1] == 0
    ctx.timing_enable([])
    got = out.cpu().numpy()
    assert np.isnan(got[M:]).all(), "rows beyond the batch were written"
    got = got[:M].astype(np.float64)

    row = np.repeat(np.arange(M), deg)
    xd = x.astype(np.float64)
    with np.errstate(all="ignore"):
        def agg(v):
            s = np.zeros((M, D))
            np.add.at(s, row, v[src])
            if model == 2:
                return (s + v[:M]) / (deg + 1)[:, None]
            return s / np.maximum(deg, 1)[:, None] if model == 0 else s
        w64 = wn.astype(np.float64)
        want = agg(xd) @ w64 + b
        size = agg(np.abs(xd)) @ np.abs(w64) + np.abs(b)
        if model != 2:
            want = want + xd[:M] @ ws.astype(np.float64)
            size = size + np.abs(xd[:M]) @ np.abs(ws.astype(np.float64))
    K = D * (1 if model == 2 else 2)
    return got, want, size * (fan + K / 8 + 8) * 2.0 ** -24


@pytest.mark.parametrize("model", [0, 1, 2])
@pytest.mark.parametrize("M,D,N,fan,cap", [
    (1, 4, 4, 3, 1), (16, 31, 64, 5, 16), (17, 33, 65, 8, 40), (40, 256, 256, 10, 96), (15, 257, 41, 15, 64), (33, 602, 47, 64, 64),
    (64, 5, 7, 2, 64), (50, 100, 130, 25, 50),                                            # few rows
    (1, 64, 256, 9, 40000), (31, 63, 256, 16, 40000), (32, 65, 129, 17, 40000), (33, 602, 172, 15, 40000), (1000, 36, 128, 33, 40000),
    (70, 4, 100, 64, 40000), (500, 130, 3, 8, 70000), (65, 96, 64, 40, 70000), (129, 101, 1, 5, 70000),    # many, by their bound
    (4096, 128, 256, 15, 5000), (3000, 4, 256, 3, 5000), (20000, 40, 64, 10, 20000), (17001, 7, 300, 2, 17001),
    (3000, 4, 256, 3, 8000), (17001, 7, 400, 2, 17001), (70, 4, 100, 20, 40000), (70, 32, 100, 64, 40000), (1000, 32, 128, 33, 40000),
    (33, 602, 47, 16, 64), (33, 128, 47, 64, 64)])
def test_layer_at_the_edges_of_its_tiles(env, model, M, D, N, fan, cap):
    got, want, bound = _run(env, M, D, N, fan, model, cap, seed=M + D + N)
    # two kernels: long lists of wide rows or of rows that are no whole lines, 257 to 384 outputs; parts of two operands' weights that do not fit
    apart = [(33, 602, 47, 64, 64), (1000, 36, 128, 33, 40000), (70, 4, 100, 64, 40000), (17001, 7, 300, 2, 17001)] + [(3000, 4, 256, 3, 5000)] * (model != 2)
    assert env["one kernel"] == ((M, D, N, fan, cap) not in apart)
    assert (np.abs(got - want) <= bound).all(), np.max(np.abs(got - want) / bound)


@pytest.mark.parametrize("model", [0, 2])
@pytest.mark.parametrize("M,D,N,cap", [(40, 100, 64, 64), (40, 100, 256, 40000), (70, 33, 64, 70000)])
def test_layer_with_numbers_that_three_parts_cannot_hold(env, model, M, D, N, cap):
    """Infinities and NaN spread as 64-bit sums spread them, numbers beyond 2^104 (whose scaled parts overflow) keep their
    value, and rows that meet none of them are as exact as ever."""
    def poke(x, ws, wn):
        x[3, 1] = np.inf
        x[5, 0] = -np.inf
        x[7, D - 1] = np.nan
        x[9, :] = 1e33
        ws[D - 1, 1] = np.inf
        wn[0, N - 1] = -np.inf
        wn[2, 2] = 2e4
    got, want, bound = _run(env, M, D, N, 6, model, cap, seed=5, poke=poke)
    assert env["one kernel"]
    assert (np.isnan(got) == np.isnan(want)).all()
    inf = np.isinf(want)
    assert (got[inf] == want[inf]).all()
    fin = np.isfinite(want)
    assert fin.any() and (np.abs(got[fin] - want[fin]) <= bound[fin]).all()


@pytest.mark.parametrize("model", [0, 2])
@pytest.mark.parametrize("everywhere", [False, True])
@pytest.mark.parametrize("D,N", [(60, 64), (60, 100), (100, 64), (100, 100), (100, 160)])
def test_tiles_of_many_rows_made_again(env, model, everywhere, D, N):
    """1,251 halves of tiles, two or three to a workgroup in the shapes of 64 columns of input and four or five in the others: first and
    second whole tiles and last halves are made again, a few of them (one row in the others') or all (a weight)."""
    M, bad = 20_011, [3, 40, 70, 130, 9_999, 20_010]

    def poke(x, ws, wn):
        for i, r in enumerate(bad):
            x[r, (7 * i) % D] = (np.inf, -np.inf, np.nan, 1e33)[i % 4]
        if everywhere:
            wn[D - 1, 1] = np.inf
    got, want, bound = _run(env, M, D, N, 3, model, M, seed=D + N, poke=poke)
    assert env["one kernel"]
    assert all(not np.isfinite(want[r]).all() or np.abs(want[r]).max() > 1e28 for r in bad)
    assert (np.isnan(got) == np.isnan(want)).all()
    inf = np.isinf(want)
    assert (got[inf] == want[inf]).all()
    fin = np.isfinite(want)
    assert fin.any(axis=1).sum() > M / 2 and (np.abs(got[fin] - want[fin]) <= bound[fin]).all()


@pytest.mark.parametrize("scale", [1e-37, 1e-30, 1e30, 1e37])
@pytest.mark.parametrize("M,D,N,cap", [(40, 100, 64, 64), (40, 100, 256, 40000)])
def test_layer_at_the_ends_of_the_range(env, scale, M, D, N, cap):
    got, want, bound = _run(env, M, D, N, 6, 0, cap, seed=8, scale=scale)
    assert env["one kernel"]
    tiny = 2.0 ** -149 * (2 * D + 8)   # products below the smallest number are lost one by one
    assert (np.abs(got - want) <= bound + tiny).all(), np.max(np.abs(got - want) / (bound + tiny))


@pytest.mark.parametrize("model", [0, 2])
@pytest.mark.parametrize("M,D,N,fan", [
    # 1,251 halves of tiles over 256 workgroups, four or five to each; the shapes' lines at 64 columns and 64 and 128 outputs
    (20_011, 64, 64, 3), (20_011, 65, 64, 3), (20_011, 64, 65, 3), (20_011, 65, 65, 3), (20_011, 64, 128, 3), (20_011, 65, 128, 3),
    (20_011, 64, 129, 3), (20_011, 65, 129, 3),
    # one half more than there are workgroups; a last half of one row; three column groups and one tile's half to each
    (4_097, 129, 100, 4), (4_097, 127, 256, 4), (8_193, 31, 41, 4), (8_193, 97, 600, 4),
    # lists around the places for their sources
    (3_000, 96, 100, 58), (3_000, 64, 128, 64)])
def test_rows_shared_out_in_halves_of_tiles(env, model, M, D, N, fan):
    got, want, bound = _run(env, M, D, N, fan, model, max(M, 9000 if fan > 4 else M), seed=M + D + N)
    assert env["one kernel"]
    assert (np.abs(got - want) <= bound).all(), np.max(np.abs(got - want) / bound)
