"""Layouts and index arithmetic of the tile passes that the compiler can check
without a GPU: the headers are compiled for the host with static assertions."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def host_compile(tmp_path, body):
    src = tmp_path / "check.hip"
    src.write_text('#include "paper_2012_01170_amd/csrc/tile_kernels.hpp"\nusing namespace sbc;\n'
                   + body)
    return subprocess.run([HIPCC, "-std=c++17", f"-I{ROOT}", "--offload-arch=gfx950",
                           "--cuda-host-only", "-fsyntax-only", str(src)],
                          capture_output=True, text=True, timeout=300)


needs_hipcc = pytest.mark.skipif(not (os.path.exists(HIPCC) or shutil.which(HIPCC)),
                                 reason="hipcc is not installed")


@needs_hipcc
def test_compact_stage_is_16_byte_aligned(tmp_path):
    """The four waves' stages lie in an array, and the compact stage moves 16
    bytes at a time: each stage starts and ends on 16 bytes."""
    r = host_compile(tmp_path, """
template <int M, int SW> constexpr bool whole() {
    using S = TileStage<M, SW, kCompact>;
    return alignof(S) % 16 == 0 && sizeof(S) % 16 == 0 && sizeof(S::v[0]) == 16;
}
static_assert(whole<8, TileShape<8, 32, kCompact>::SW>(), "M 8, 32 rows");
static_assert(whole<8, TileShape<8, 64, kCompact>::SW>(), "M 8, 64 rows");
static_assert(whole<10, TileShape<10, 32, kCompact>::SW>(), "M 10, 32 rows");
static_assert(whole<10, TileShape<10, 64, kCompact>::SW>(), "M 10, 64 rows");
static_assert(whole<8, DwShape<8, 2, kCompact>::SW>(), "M 8, weight gradient");
static_assert(whole<8, DwShape<8, 4, kCompact>::SW>(), "M 8, weight gradient");
static_assert(whole<10, DwShape<10, 4, kCompact>::SW>(), "M 10, weight gradient");
""")
    assert r.returncode == 0, r.stderr


@needs_hipcc
def test_row_bounds_stay_in_range(tmp_path):
    """The row pointer a lane reads, up to the last rows of the largest pattern
    (in a constant expression an overflow of int32 is an error)."""
    r = host_compile(tmp_path, """
constexpr int32_t n = 2147483647;
static_assert(row_at(0, 0, 1) == 0 && row_at(0, 1, 1) == 1 && row_at(0, 16, 1) == 1, "one row");
static_assert(row_at(48, 16, 65) == 64 && row_at(64, 16, 65) == 65, "a ragged tile");
static_assert(row_at(n - 15, 16, n) == n && row_at(n - 63 + 48, 16, n) == n, "the last tile");
static_assert(row_at(n - 16, 15, n) == n - 1 && row_at(n, 16, n) == n, "the last row");
""")
    assert r.returncode == 0, r.stderr
