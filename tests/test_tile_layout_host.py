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
