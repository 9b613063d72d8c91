"""The input layer as one kernel with its weights in registers (DCI_OPT_INPUT_LAYER 2), with several 32-row blocks to a
workgroup: more than 8,192 rows on 256 compute units, where a block's rows are added up between the matrix instructions of the
block before it.  Every source of a row must be in its mean, however short the contraction is.  The bound: a mean of up to 15
rows and a contraction of 2 D products, added one after the other in fp32."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [16, 32, 36, 64, 68, 100, 104, 128])
def test_every_source_is_added_in_every_block(D):
    import paper_2503_01281_amd as dci
    ctx = dci.Context(0)
    M, N, fan = 20_001, 256, 15
    rng = np.random.default_rng(D)
    blk = dci.Blocks(ctx, 10**7, M, (fan,))
    deg = rng.integers(0, fan + 1, M)
    indptr = np.concatenate([[0], deg.cumsum()])
    src = rng.integers(0, M, indptr[-1])
    blk.counts.zero_()
    blk.counts[0] = blk.counts[1] = M
    blk.blk_indptr[0][:M + 1] = torch.from_numpy(indptr).cuda()
    blk.blk_src[0][:len(src)] = torch.from_numpy(src.astype(np.int32)).cuda()
    x = rng.standard_normal((M, D)).astype(np.float32)
    ws, wn = (rng.uniform(-1, 1, (2, D, N)) * np.sqrt(6 / (D + N))).astype(np.float32)
    b = rng.uniform(-0.1, 0.1, N).astype(np.float32)
    dev = lambda a: torch.from_numpy(a).cuda()
    x_dev = torch.zeros(blk.cap_nodes[1], D, dtype=torch.float32, device="cuda")
    x_dev[:M] = dev(x)
    out = torch.empty(blk.cap_nodes[0], N, dtype=torch.float32, device="cuda")
    ctx.set_option(dci.DCI_OPT_INPUT_LAYER, 2)
    dci.dci_sage_forward(ctx, blk, x_dev, [dev(ws)], [dev(wn)], [dev(b)], out)
    ctx.sync()
    x64, row = torch.from_numpy(x).double(), torch.from_numpy(np.repeat(np.arange(M), deg))

    def layer(v, a, c):
        m = torch.zeros(M, D, dtype=torch.float64).index_add_(0, row, v[torch.from_numpy(src)])
        return v @ a + m / torch.from_numpy(np.maximum(deg, 1))[:, None] @ c
    w = [torch.from_numpy(a).double() for a in (ws, wn)]
    want = layer(x64, *w) + torch.from_numpy(b).double()
    bound = (layer(x64.abs(), *[a.abs() for a in w]) + 0.1) * (2 * D + fan + 2) * 2.0 ** -24
    assert bool(((out[:M].cpu().double() - want).abs() <= bound).all())
