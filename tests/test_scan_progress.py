"""Tiles of the frontier scan that are numbered by their workgroup (CPU: the header's own constants, compiled for the host): however many
compute units the process sees, the workgroups of all scans that may be on the card together have a place each."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_tiles_without_tickets_all_have_a_place(tmp_path):
    from paper_2503_01281_amd import build
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc here")
    src = tmp_path / "places.hip"
    src.write_text("""#include "dci_internal.h"
constexpr bool places(int cus) {  // a scan of one tile waits for nobody
  return dci::unticketed_tiles(cus) <= 1 || (int)dci::unticketed_tiles(cus) * 64 <= 4 * cus;
}
constexpr bool all() {
  for (int cus = 1; cus <= 512; ++cus)
    if (!places(cus)) return false;
  return true;
}
static_assert(all(), "16 processes of four queues each, four workgroups to a compute unit");
static_assert(dci::kRelabelPerCu == 4 && dci::unticketed_tiles(256) == 16 && dci::unticketed_tiles(32) == 2, "");
""")
    r = subprocess.run([hipcc, "--cuda-host-only", "-fsyntax-only", "-std=c++17", "-x", "hip", "-I", os.path.join(ROOT, "include"),
                        "-I", build.CSRC, str(src)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
