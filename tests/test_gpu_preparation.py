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
