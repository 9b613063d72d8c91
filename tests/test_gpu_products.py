"""What the default layers' products (fp32 operands in three bf16 parts) carry.

A product by itself: the part sums' own rounding is below 6 x 2^-23 x 2^-7 of it, what is left out below 2^-33, and the addition
of the two sums rounds it once, so it is within 1.1 x 2^-24 (fp32 products: 2^-24).  Sums: against 64 bits no worse than the
kernels that multiply with the fp32 instructions, for inputs of both signs and of one, for numbers whose parts are as large
as they can be, in contractions of a few columns and of many."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import paper_2503_01281_amd as dci
    return {"dci": dci, "ctx": dci.Context(0)}


KINDS = {  # (rows, weights) of a generator; "parts": numbers whose second and third parts are near their bounds
    "normal": (lambda g, *s: torch.randn(*s, generator=g), lambda g, k, n: (torch.rand(k, n, generator=g) * 2 - 1) * (6 / (k + n)) ** 0.5),
    "one sign": (lambda g, *s: 1 + torch.rand(*s, generator=g),) * 2,
    "near one": (lambda g, *s: 1 + torch.rand(*s, generator=g) / 64,) * 2,
    "parts": (lambda g, *s: torch.tensor(1 + 2.0 ** -8 - 2.0 ** -17) + torch.randint(0, 4, s, generator=g) * 2.0 ** -23,) * 2,
}


def _layer(env, kind, M, cap, D, N, model, one_product):
    """(x, self weights, neighbour weights, sources of one neighbour per row or None, result of the default, of option 1)"""
    dci, ctx = env["dci"], env["ctx"]
    g = torch.Generator().manual_seed(1000 * D + M)
    blk = dci.Blocks(ctx, 10**7, cap, (1,))
    fx, fw = KINDS[kind]
    x = fx(g, M, D).float()
    src = torch.randint(0, M, (M,), generator=g, dtype=torch.int32)
    blk.blk_indptr[0].zero_()
    if one_product:
        at = torch.randint(0, D, (M,), generator=g)
        x = torch.zeros_like(x).scatter_(1, at[:, None], x.gather(1, at[:, None]))
    else:
        blk.blk_indptr[0][:M + 1] = torch.arange(M + 1).cuda()
        blk.blk_src[0][:M] = src.cuda()
    blk.counts.zero_()
    blk.counts[0] = blk.counts[1] = M
    ws, wn = (fw(g, D, N).float() for _ in range(2))
    x_dev = torch.zeros(max(M, blk.cap_nodes[0]), D, device="cuda")
    x_dev[:M] = x.cuda()
    got = []
    for option in (0, 1):
        out = torch.empty(blk.cap_nodes[0], N, device="cuda")
        ctx.set_option(dci.DCI_OPT_LINEAR_KERNEL, option)
        try:
            dci.dci_gnn_forward(ctx, blk, x_dev, model, None if model == 2 else [ws.cuda()], [wn.cuda()], [torch.zeros(N, device="cuda")], out)
            ctx.sync()
        finally:
            ctx.set_option(dci.DCI_OPT_LINEAR_KERNEL, 0)
        got.append(out[:M].cpu().double())
    return x.double(), ws.double(), wn.double(), None if one_product else src.long(), got


@pytest.mark.parametrize("kind", ["normal", "one sign", "parts"])
@pytest.mark.parametrize("model", [0, 2])
@pytest.mark.parametrize("M,cap,N", [(500, 512, 64), (4000, 40000, 64), (4000, 40000, 128), (4000, 40000, 256)])
def test_a_product_by_itself_is_as_exact_as_in_fp32(env, kind, model, M, cap, N):
    for D in (4, 33, 70, 602):
        x, ws, wn, _, (got, _) = _layer(env, kind, M, cap, D, N, model, True)
        want = x @ (wn if model == 2 else ws)
        off = ((got - want).abs() / want.abs().clamp(min=1e-30)).max().item() * 2.0 ** 24
        assert off <= 1.1, (D, off)


@pytest.mark.parametrize("kind", list(KINDS))
@pytest.mark.parametrize("M,cap,N", [(500, 512, 64), (4000, 40000, 256)])
def test_sums_are_no_worse_than_the_fp32_instructions(env, kind, M, cap, N):
    for D in (4, 5, 6, 8, 12, 16, 24, 32, 48, 64, 100, 128, 256, 602):
        x, ws, wn, src, got = _layer(env, kind, M, cap, D, N, 0, False)
        want = x @ ws + x[src] @ wn
        size = x.abs() @ ws.abs() + x[src].abs() @ wn.abs()
        off = [(v - want) / size * 2.0 ** 24 for v in got]
        rms, top = [float(v.pow(2).mean().sqrt()) for v in off], [float(v.abs().max()) for v in off]
        print(f"{kind} {M} x {D} x {N}: rms {rms[0]:.3f} / {rms[1]:.3f}, largest {top[0]:.2f} / {top[1]:.2f} (2^-24)")
        assert rms[0] <= rms[1] and top[0] <= top[1], (D, rms, top)
