"""The route that the sizes of a convolution choose, on the host: the measured
sides of the line, and that every call finds its workspace."""
import pytest
import torch

from paper_2012_01170_amd import _lib as L
from paper_2012_01170_amd import ops


@pytest.fixture(scope="module")
def lib():
    return L.lib()


# rows, entries a row, M, C_in, C_out, the gather and contraction in one kernel
# (measured us: that kernel, the separate ones)
@pytest.mark.parametrize("n,deg,M,ci,co,fused", [
    (32768, 6, 8, 128, 128, True),      # 70, 166
    (32768, 6, 8, 512, 128, True),      # 236, 405
    (32768, 20, 8, 64, 8, True),        # 51, 108
    (32768, 20, 8, 512, 8, False),      # 322, 128
    (32768, 20, 4, 512, 8, False),      # 273, 96
    (32768, 20, 10, 512, 8, False),     # 389, 163
    (4096, 16, 8, 512, 8, False),       # 117, 35
    (4096, 16, 8, 512, 64, False),      # 120, 57
    (32768, 6, 4, 64, 8, True),         # 23, 42
])
def test_routes_follow_the_measured_times(lib, n, deg, M, ci, co, fused):
    assert ops.conv_plan(n, n, n * deg, M, ci, co)["forward_fused"] == fused
    # an explicit order is kept, and a tile pass is a gather-first one
    p = ops.conv_plan(n, n, n * deg, M, ci, co, order="gemm_first")
    assert p["forward_order"] == p["backward_order"] == "gemm_first" and not p["forward_fused"]
    p = ops.conv_plan(n, n, n * deg, M, ci, co, order="spmm_first")
    assert p["forward_order"] == p["backward_order"] == "spmm_first"


def test_up_sampling_contracts_first(lib):
    assert ops.conv_plan(32768, 8192, 160_000, 8, 128, 64)["forward_order"] == "gemm_first"


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_every_shape_has_a_workspace(lib, dtype):
    """Also at the sizes where nothing is gathered or a tile is all there is; where
    the forward runs as separate kernels it holds the smaller intermediate."""
    code = L.SBC_BF16 if dtype == torch.bfloat16 else L.SBC_F32
    for M in (4, 8, 10, 16, 24, 32):
        for ci, co in ((8, 8), (33, 40), (128, 128), (512, 8), (8, 512), (512, 512)):
            for n in (1, 100, 4096, 50_000):
                for deg in (0, 1, 6, 40):
                    size = lib.sbc_conv_workspace_size(n, n, n * deg, M, ci, co, code,
                                                       L.SBC_ORDER_AUTO)
                    assert size > 0
                    if ops.conv_plan(n, n, n * deg, M, ci, co, dtype=dtype)["forward_fused"]:
                        continue
                    assert size >= n * M * min(ci, co) * 4


def test_intermediates_past_2_to_the_31_stay_on_the_tile_pass(lib):
    """Rows times M times channels: the separate kernels compete below 2^31 (here
    for the gradients, whose workspace is the larger)."""
    n, M, c = (1 << 31) // (4 * 512), 4, 512
    size = lambda rows: lib.sbc_conv_workspace_size(rows, rows, rows * 40, M, c, c, L.SBC_F32,
                                                    L.SBC_ORDER_AUTO)
    assert size(n - 1) >= 4 * (n - 1) * M * c
    assert size(n) < 1 << 30 and ops.conv_plan(n, n, n * 40, M, c, c)["forward_fused"]
