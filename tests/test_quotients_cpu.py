"""Quotients by a state count as a 32-bit multiply and a shift: exact over the entries that
a kernel divides, and a build whose tiles pass the bound is refused.
"""
import os
import re
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "paper_1909_11469_amd", "csrc", "bp_internal.h")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def _constant(name):
    m = re.search(rf"(?:#define\s+{name}|constexpr int {name} =)\s+(\d+)", open(HEADER).read())
    return int(m.group(1))


@pytest.mark.parametrize("kmin,kmax,limit", [
    (3, _constant("kMaxK"),
     _constant("BP_TILE_FLOATS_GENERIC") + _constant("kPairsUnroll") * _constant("BP_BLOCK")),
    (2, _constant("kMaxKRagged"), _constant("BP_RAGGED_FLAT"))])
def test_every_quotient_is_exact(kmin, kmax, limit):
    i = np.arange(limit, dtype=np.uint32)
    for K in range(kmin, kmax + 1):
        magic = np.uint32((1 << 20) // K + 1)
        assert np.array_equal((i * magic) >> np.uint32(20), i // np.uint32(K)), K


def test_the_bound_is_where_the_quotient_breaks():
    # K = 3: the product wraps at 12,288
    magic = np.uint32((1 << 20) // 3 + 1)
    i = np.array([12287, 12288], dtype=np.uint32)
    assert list((i * magic) >> np.uint32(20)) == [4095, 0]


@pytest.mark.parametrize("define,ok", [("BP_TILE_FLOATS_GENERIC=8192", True),
                                       ("BP_TILE_FLOATS_GENERIC=12288", False),
                                       ("BP_RAGGED_FLAT=8192", True),
                                       ("BP_RAGGED_FLAT=8193", False)])
def test_a_build_past_the_bound_is_refused(define, ok):
    r = subprocess.run([HIPCC, "-std=c++17", "--offload-arch=gfx950", "--offload-host-only",
                        "-fsyntax-only", "-x", "hip", "-D" + define, HEADER],
                       capture_output=True, text=True)
    assert (r.returncode == 0) == ok, r.stderr
    assert ok or "exact quotients" in r.stderr
