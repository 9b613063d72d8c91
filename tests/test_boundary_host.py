"""Host-side checks of the C boundary that need no GPU: the library loads, exports every symbol
the header declares, and its pure host logic (bounds, workspace sizes, argument checks) behaves."""
import ctypes as C
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    import paper_2503_01281_amd as dci
    if not os.path.exists(dci.library_path()):
        from paper_2503_01281_amd import build
        build.build()
    return dci.load_library()


def test_every_declared_symbol_is_exported(lib):
    header = open(os.path.join(ROOT, "include", "dci.h")).read()
    header = re.sub(r"/\*.*?\*/", "", header, flags=re.S)
    names = sorted(set(re.findall(r"\b(dci_[a-z_0-9]+)\s*\(", header)))
    assert {"dci_presample_count", "dci_fill_caches", "dci_sample_khop", "dci_gather_features",
            "dci_sage_forward", "dci_create", "dci_destroy", "dci_sync", "dci_last_error"} <= set(names)
    for n in names:
        assert hasattr(lib, n), f"{n} is declared in include/dci.h but not exported by libdci.so"


def test_blocks_bounds():
    import paper_2503_01281_amd as dci
    assert dci.blocks_bounds(232965, 1024, [5, 10, 15]) == ([1024, 6144, 67584, 233989], [5120, 61440, 1013760])
    assert dci.blocks_bounds(16384, 256, [5, 10]) == ([256, 1536, 16640], [1280, 15360])
    assert dci.blocks_bounds(10, 0, [3]) == ([0, 0], [0])
    for bad in ([], [0], [65], [5] * 9):
        with pytest.raises(dci.DciError):
            dci.blocks_bounds(1000, 10, bad)
    with pytest.raises(dci.DciError) as e:           # a bound at or above 2^31
        dci.blocks_bounds(2**31 - 1, 2**26, [64, 64])
    assert e.value.code == -4


def test_workspace_queries_grow_with_the_problem(lib):
    f3 = (C.c_int32 * 3)(5, 10, 15)
    small = lib.dci_sample_workspace_bytes(232965, 256, f3, 3)
    big = lib.dci_sample_workspace_bytes(232965, 1024, f3, 3)
    assert 0 < small < big
    assert lib.dci_sample_workspace_bytes(232965, 1024, (C.c_int32 * 1)(0), 1) == 0      # invalid fan-out
    assert 0 < lib.dci_fill_workspace_bytes(1000) < lib.dci_fill_workspace_bytes(10**6)
    assert lib.dci_fill_workspace_bytes(0) == 0
    rows = (C.c_int64 * 8)(1024, 6144, 67584, 0, 0, 0, 0, 0)
    dims = (C.c_int32 * 4)(602, 256, 256, 41)
    need = lib.dci_sage_workspace_bytes(rows, 3, dims)
    assert need >= 67584 * 602 * 4 + 2 * 67584 * 256 * 4


def test_fill_workspace_stays_what_its_arrays_take(lib):
    """Five arrays of a word per node, the sort's histograms and scan sums, two counter totals: nothing of a size of its
    own, so a workspace that a caller sized once keeps being enough."""
    up = lambda n: -(-n // 256) * 256
    sort = lambda n: 4 * up(4 * n) + up(1024 * -(-n // 4096)) + up(8 * (-(-max(n, 256 * -(-n // 4096)) // 2048) + 1))
    for n in (1, 1_000, 2_449_029):
        fill = 256 + up(4 * n) + sort(n)
        assert lib.dci_fill_workspace_bytes(n) == fill
        e = 10 * n
        assert lib.dci_fill_elements_workspace_bytes(n, e) == fill + up(8 * (n + 1)) + up(8 * e) + 2 * up(4 * e) + sort(e)


def test_static_scratch_size_query(lib):
    """The no-allocation sampler's size query (host arithmetic only): a Medium-sized batch fits the
    static array, a Large-sized one does not, invalid fan-outs give 0."""
    lib.dci_sample_khop_scratch_bytes.restype = C.c_size_t
    f3 = (C.c_int32 * 3)(5, 10, 15)
    limit = 32 << 20
    assert 0 < lib.dci_sample_khop_scratch_bytes(232965, 1024, f3, 3) <= limit
    assert lib.dci_sample_khop_scratch_bytes(2449029, 4096, f3, 3) > limit
    assert lib.dci_sample_khop_scratch_bytes(232965, 1024, (C.c_int32 * 1)(65), 1) == 0
    assert lib.dci_sample_khop_static(None, None, None, None, 0, 0, None, 0, 0, None, None) == -1


def test_null_context_and_missing_gpu_are_errors_not_crashes(lib):
    assert lib.dci_sync(None) == -1
    assert lib.dci_set_workspace(None, None, 0) == -1
    assert lib.dci_last_error(None) == b"null context"
    assert lib.dci_sample_khop(None, None, None, None, 0, 0, None, 0, 0, None, None) == -1
    assert lib.dci_gather_features(None, None, None, None, 0, None, None, None) == -1
    assert lib.dci_fill_caches(None, None, None, None, None, 0, 0, 0, 0, None, None, None, None, None) == -1
    assert lib.dci_create(None, 0, None, None, 0) == -1
    import torch
    if not torch.cuda.is_available():
        h = C.c_void_p()
        assert lib.dci_create(C.byref(h), 0, None, None, 0) == -3      # no device: a HIP error, reported
        assert not h.value


def test_the_binding_has_no_fallback():
    """The Python layer only marshals arguments: it must not import the oracle or implement the path."""
    for fn in ("binding.py", "__init__.py"):
        src = open(os.path.join(ROOT, "paper_2503_01281_amd", fn)).read()
        assert "oracle" not in src and "numpy" not in src


def test_a_workspace_grows_for_a_need_within_its_alignment():
    """What the library is told it has is 256 bytes less than what was allocated; a need between the two asks for a new one."""
    import torch

    import paper_2503_01281_amd as dci

    class Lib:
        told = []

        def dci_sync(self, h):
            return 0

        def dci_set_workspace(self, h, base, nbytes):
            assert base % 256 == 0
            self.told.append(nbytes)
            return 0

        def dci_destroy(self, h):
            pass

    ctx = dci.Context.__new__(dci.Context)
    ctx.lib, ctx._h, ctx._ws, ctx.device = Lib(), C.c_void_p(), None, torch.device("cpu")
    for need in (1000, 1000, 999, 1001, 1256, 1257, 5000):
        ctx.ensure_workspace(need)
        assert Lib.told[-1] >= need
    assert len(Lib.told) == 5 and Lib.told[0] == 1000
