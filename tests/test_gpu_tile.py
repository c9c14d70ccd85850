"""The tile passes of the convolution (gather, split into bf16 parts and
contraction in one kernel, any channel counts) under AUTO: against the oracle
and against the separate-kernel route (order "gemm_first"), at the edges of
their tiles: rows, slices of 32 channels, column blocks of 16, chunks of 64 and
128 channels, rows longer than the stage, one row, no edges.  AUTO gives long
rows, wide chunks and many basis functions at these row counts to the separate
kernels; test_gpu_routes.py takes those through the tile passes at sizes where
it does not, and checks by the launches which ran."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from tests import gpu_common as G

pytestmark = pytest.mark.gpu

P, E = workloads.small_points, workloads.small_events
CASES = {
    "c8": lambda: P(seed=40, c_in=8, c_out=8),
    "odd_rows": lambda: P(seed=41, n_clouds=1, n=65, c_in=33, c_out=31),
    "mono4_chunks": lambda: P(seed=42, basis=workloads.BASIS_MONO4, c_in=130, c_out=65),
    "wide_out": lambda: P(seed=43, n_out=33, c_in=32, c_out=129),
    "down": lambda: P(seed=44, n_out=40, c_in=24, c_out=96),
    "weighted": lambda: P(seed=45, basis=workloads.BASIS_WMONO10, c_in=40, c_out=72),
    "weighted_wide": lambda: P(seed=46, basis=workloads.BASIS_WMONO10, c_in=68, c_out=20, n_out=31),
    "bf16_odd": lambda: P(seed=47, c_in=17, c_out=48, dtype="bf16"),
    "bf16_wide": lambda: P(seed=48, basis=workloads.BASIS_MONO4, c_in=64, c_out=132, dtype="bf16"),
    "bf16_weighted": lambda: P(seed=49, basis=workloads.BASIS_WMONO10, c_in=36, c_out=68,
                               dtype="bf16"),
    # whole clouds as neighbourhoods: rows of 200 entries and more
    "long_rows": lambda: P(seed=50, n_clouds=2, n=200, radius=3.0, k_cap=0, c_in=20, c_out=36),
    "long_rows_weighted": lambda: P(seed=51, n_clouds=2, n=210, radius=3.0, k_cap=0, c_in=12,
                                    c_out=12, basis=workloads.BASIS_WMONO10),
    "one_point": lambda: P(seed=52, n_clouds=1, n=1, c_in=16, c_out=16),
    "events": lambda: E(seed=40, n=2049, c=48),
    "events_odd_bf16": lambda: E(seed=41, n=1500, c=21, dtype="bf16"),
    "decays2": lambda: E(seed=42, n=1100, c=20, n_decays=2),
    "decays3": lambda: E(seed=43, n=1100, c=40, n_decays=3),
    "decays4": lambda: E(seed=44, n=1100, c=9, n_decays=4),
    # 64-row tiles: two blocks per CU of them
    "tall": lambda: P(seed=53, n_clouds=24, n=1024, radius=0.1, c_in=12, c_out=12,
                      basis=workloads.BASIS_MONO4),
}


def _assert_tile_forward(n, nnz, M, ci, co, dtype=torch.float32):
    """The sizes are ones that the tile pass is chosen for."""
    assert G.sbc.conv_plan(n, n, nnz, M, ci, co, dtype=dtype)["forward_fused"]


def _pattern(w):
    if w["kind"] == "points":
        rp, ci = oracle.points_csr(w["x_in"], w["in_splits"], w["x_out"], w["out_splits"],
                                   w["radius"], w["k_cap"])
        v = oracle.basis.point_values(w["basis"], w["x_in"], w["x_out"], rp, ci, w["radius"],
                                      w["M"])
    else:
        rp, ci = oracle.events_csr(w["px"], w["py"], w["t"], w["window"], 1, w["width"],
                                   w["height"])
        v = oracle.basis.event_values(w["basis"], w["px"], w["py"], w["t"], rp, ci, w["tau"],
                                      w.get("decays"))
    return rp, ci, v


@pytest.mark.parametrize("name", list(CASES))
def test_tile_passes(name):
    print(f"[tile] {name}", flush=True)
    w = CASES[name]()
    rp, ci, v = _pattern(w)
    t = G.to_device(w)
    csr = G.search(w, t)
    geo = G.geometry(w, t)
    csc = G.sbc.csr_transpose(csr)
    Y_ref = oracle.conv.forward(rp, ci, v, w["F"], w["W"])
    dF_ref, dW_ref = oracle.conv.backward(rp, ci, v, w["F"], w["W"], w["dY"], w["n_in"])
    # float32 sums on every route: bf16 inputs are exact in them, so the float32
    # tolerance holds for both types
    tol = G.TOL_F32
    vd = torch.from_numpy(np.ascontiguousarray(v, dtype=np.float32)).to(G.DEV)
    if vd.numel() == 0:
        vd = None
    for order in ("auto", "gemm_first"):
        for values in (None, vd):
            g = geo if values is None else None
            if g is None and values is None:
                continue
            Y = G.sbc.conv_forward(csr, t["F"], t["W"], geometry=g, v=values, order=order)
            dF, dW = G.sbc.conv_backward(csr, csc, t["F"], t["W"], t["dY"], geometry=g, v=values,
                                         order=order)
            assert G.row_error(Y.cpu().numpy(), Y_ref) < tol, (order, values is None)
            assert G.row_error(dF.cpu().numpy(), dF_ref) < tol, (order, values is None)
            assert G.norm_error(dW.cpu().numpy(), dW_ref) < tol, (order, values is None)


def test_tile_passes_without_edges():
    """Rows without entries are exact zeros, and so is the weight gradient."""
    n, M, ci, co = 70, 8, 40, 24
    z = lambda *s: torch.randn(s, device=G.DEV)
    csr = G.sbc.CSR(torch.zeros(n + 1, dtype=torch.int32, device=G.DEV),
                    torch.zeros(1, dtype=torch.int32, device=G.DEV), n, n, 0)
    csc = G.sbc.csr_transpose(csr)
    x = z(n, 3)
    geo = G.sbc.Geometry("mono8", radius=0.1, x_in=x, x_out=x)
    F, W, dY = z(n, ci), z(M, ci, co), z(n, co)
    assert not bool(G.sbc.conv_forward(csr, F, W, geometry=geo).any())
    dF, dW = G.sbc.conv_backward(csr, csc, F, W, dY, geometry=geo)
    assert not bool(dF.any()) and not bool(dW.any())


@pytest.mark.parametrize("bad", [float("inf"), float("-inf"), float("nan")])
def test_tile_passes_keep_infinities(bad):
    """An infinite or NaN feature shows where float32 products show it (an
    infinity stays one where nothing of the opposite sign meets it) and leaves
    the rows that do not gather it as they are, bit for bit."""
    n, ci, co = 96, 36, 20
    rp = torch.arange(n + 1, dtype=torch.int32, device=G.DEV)
    idx = torch.arange(n, dtype=torch.int32, device=G.DEV)
    csr = G.sbc.CSR(rp, idx, n, n, n)
    csc = G.sbc.csr_transpose(csr)
    gen = torch.Generator(device=G.DEV)
    gen.manual_seed(5)
    z = lambda *s: torch.rand(s, generator=gen, device=G.DEV) + 0.5
    v = z(n, 4)
    F, W, dY = z(n, ci), z(4, ci, co), z(n, co)
    Y0 = G.sbc.conv_forward(csr, F, W, v=v)
    dF0, _ = G.sbc.conv_backward(csr, csc, F, W, dY, v=v)
    F2, dY2 = F.clone(), dY.clone()
    F2[17, 5] = bad
    dY2[40, 3] = bad
    Y = G.sbc.conv_forward(csr, F2, W, v=v)
    dF, dW = G.sbc.conv_backward(csr, csc, F2, W, dY2, v=v)
    same = lambda x: bool(torch.isnan(x).all()) if bad != bad else bool((x == bad).all())
    keep = torch.arange(n, device=G.DEV)
    assert same(Y[17]) and torch.equal(Y[keep != 17], Y0[keep != 17])
    assert same(dF[40]) and torch.equal(dF[keep != 40], dF0[keep != 40])
    assert same(dW[:, 5, :]) and same(dW[:, :, 3])
    rest = torch.ones((ci, co), dtype=torch.bool, device=G.DEV)
    rest[5, :] = False
    rest[:, 3] = False
    assert bool(torch.isfinite(dW[:, rest]).all())


@pytest.mark.parametrize("bits", [0x7F800001, -0x7FFFFE, 0x7FC00000], ids=["low", "minus_low", "quiet"])
def test_tile_passes_keep_every_nan(bits):
    """A NaN is one by its bits: also one whose payload lies below the upper 16
    bits, as a weight, a feature and an upstream gradient."""
    n, ci, co = 96, 36, 20
    _assert_tile_forward(n, n, 4, ci, co)
    idx = torch.arange(n + 1, dtype=torch.int32, device=G.DEV)
    csr = G.sbc.CSR(idx, idx[:n].contiguous(), n, n, n)
    csc = G.sbc.csr_transpose(csr)
    gen = torch.Generator(device=G.DEV)
    gen.manual_seed(6)
    z = lambda *s: torch.rand(s, generator=gen, device=G.DEV) + 0.5
    v = z(n, 4)

    def poisoned(x, *at):
        y = x.clone()
        y.view(torch.int32)[at] = bits
        assert bool(torch.isnan(y[at]))
        return y

    F, W, dY = z(n, ci), z(4, ci, co), z(n, co)
    nan = lambda x: bool(torch.isnan(x).all())
    Wn = poisoned(W, 2, 7, 3)
    Y = G.sbc.conv_forward(csr, F, Wn, v=v)
    dF, _ = G.sbc.conv_backward(csr, csc, F, Wn, dY, v=v)
    assert nan(Y[:, 3]) and bool(torch.isfinite(Y[:, :3]).all())
    assert nan(dF[:, 7]) and bool(torch.isfinite(dF[:, :7]).all())
    Fn, dYn = poisoned(F, 17, 5), poisoned(dY, 40, 3)
    Y = G.sbc.conv_forward(csr, Fn, W, v=v)
    dF, dW = G.sbc.conv_backward(csr, csc, Fn, W, dYn, v=v)
    assert nan(Y[17]) and nan(dF[40]) and nan(dW[:, 5, :]) and nan(dW[:, :, 3])


@pytest.mark.parametrize("k", [0, 100, 114, 122])
def test_tile_passes_on_tiny_operands(k):
    """Operands of size 2^-k on either side: 2^-134 of an operand is lost to the
    parts' smallest value, beside the float32 sums' 1e-6 (positive terms only,
    so errors do not grow by cancellation)."""
    n, ci, co = 96, 36, 20
    _assert_tile_forward(n, n, 4, ci, co)
    idx = torch.arange(n + 1, dtype=torch.int32, device=G.DEV)
    csr = G.sbc.CSR(idx, idx[:n].contiguous(), n, n, n)
    csc = G.sbc.csr_transpose(csr)
    gen = torch.Generator(device=G.DEV)
    gen.manual_seed(7)
    z = lambda *s: torch.rand(s, generator=gen, device=G.DEV) + 0.5
    v = torch.ones(n, 4, device=G.DEV)
    F, W, dY, s = z(n, ci), z(4, ci, co), z(n, co), 2.0 ** -k
    tol = 1e-6 + 2.0 ** -134 / (0.5 * s)

    def check(got, ref):
        assert float(((got.double() - ref).abs() / ref).max()) < tol

    d, Wsum = torch.float64, W.to(torch.float64).sum(0)
    check(G.sbc.conv_forward(csr, F * s, W, v=v), (F * s).to(d) @ Wsum)
    check(G.sbc.conv_forward(csr, F, W * s, v=v), F.to(d) @ (Wsum * s))
    dF, dW = G.sbc.conv_backward(csr, csc, F, W, dY * s, v=v)
    check(dF, (dY * s).to(d) @ Wsum.t().contiguous())
    check(dW[1], F.to(d).t().contiguous() @ (dY * s).to(d))


# Patterns of two blocks of 64 rows per CU and more, where the mean number of
# entries chooses the tile's height (10 a row, 16 for float32 and more than 64
# columns; event bases: 64 rows always): (rows short, workload).
_BIG = dict(n_clouds=33, n=1000, radius=0.5)
TALL = {
    "f32_short": (True, lambda: P(seed=90, k_cap=6, c_in=20, c_out=33, **_BIG)),
    "f32_long": (False, lambda: P(seed=90, k_cap=14, c_in=20, c_out=33, **_BIG)),
    "f32_ten": (True, lambda: P(seed=91, k_cap=10, c_in=12, c_out=12, **_BIG)),
    "f32_eleven": (False, lambda: P(seed=91, k_cap=11, c_in=12, c_out=12, **_BIG)),
    "f32_wide_short": (True, lambda: P(seed=92, k_cap=14, c_in=36, c_out=72, **_BIG)),
    "f32_wide_long": (False, lambda: P(seed=92, k_cap=18, c_in=36, c_out=72, **_BIG)),
    "bf16_pieces_short": (True, lambda: P(seed=93, k_cap=5, c_in=40, c_out=24, dtype="bf16", **_BIG)),
    "bf16_pieces_long": (False, lambda: P(seed=93, k_cap=13, c_in=40, c_out=24, dtype="bf16", **_BIG)),
    "bf16_odd_wide_short": (True, lambda: P(seed=94, k_cap=5, c_in=21, c_out=70, dtype="bf16", **_BIG)),
    "bf16_odd_wide_long": (False, lambda: P(seed=94, k_cap=12, c_in=21, c_out=70, dtype="bf16", **_BIG)),
    "weighted_short": (True, lambda: P(seed=95, k_cap=5, c_in=16, c_out=64,
                                       basis=workloads.BASIS_WMONO10, **_BIG)),
    "weighted_long": (False, lambda: P(seed=95, k_cap=12, c_in=16, c_out=64,
                                       basis=workloads.BASIS_WMONO10, **_BIG)),
    "mono4_long": (False, lambda: P(seed=96, k_cap=15, c_in=68, c_out=17,
                                    basis=workloads.BASIS_MONO4, **_BIG)),
    "events": (None, lambda: E(seed=97, n=33000, width=128, height=96, c=48)),
    "events_bf16_wide": (None, lambda: E(seed=98, n=33000, width=96, height=96, c=72, dtype="bf16")),
    "events_long": (None, lambda: E(seed=99, n=33000, width=64, height=40, c=20)),
}


@pytest.mark.parametrize("name", list(TALL))
def test_tile_height(name):
    short, make = TALL[name]
    w = make()
    print(f"[tile height] {name}", flush=True)
    rp, ci, v = _pattern(w)
    mean = len(ci) / w["n_out"]
    assert w["n_out"] // 64 >= 512
    _assert_tile_forward(w["n_out"], len(ci), w["M"], w["C_in"], w["C_out"],
                         torch.bfloat16 if w["dtype"] == "bf16" else torch.float32)
    wide = w["dtype"] == "f32" and w["C_out"] > 64
    if short is not None:
        assert short == (mean <= (16 if wide else 10))
    t = G.to_device(w)
    csr = G.search(w, t)
    geo = G.geometry(w, t)
    csc = G.sbc.csr_transpose(csr)
    Y_ref = oracle.conv.forward(rp, ci, v, w["F"], w["W"])
    dF_ref, dW_ref = oracle.conv.backward(rp, ci, v, w["F"], w["W"], w["dY"], w["n_in"])
    vd = torch.from_numpy(np.ascontiguousarray(v, dtype=np.float32)).to(G.DEV)
    for geometry, values in ((geo, None), (None, vd)):
        Y = G.sbc.conv_forward(csr, t["F"], t["W"], geometry=geometry, v=values)
        dF, dW = G.sbc.conv_backward(csr, csc, t["F"], t["W"], t["dY"], geometry=geometry, v=values)
        assert G.row_error(Y.cpu().numpy(), Y_ref) < G.TOL_F32
        assert G.row_error(dF.cpu().numpy(), dF_ref) < G.TOL_F32
        assert G.norm_error(dW.cpu().numpy(), dW_ref) < G.TOL_F32


@pytest.mark.parametrize("n,c_out", [(40, 128), (40, 33), (2048, 128), (4096, 128), (4160, 128),
                                     (8192, 64), (8193, 64), (300, 300)])
def test_tile_columns(n, c_out):
    """Blocks of 32, 64 and 128 columns, chosen by the rows: every column of
    every row, last blocks included."""
    print(f"[tile columns] {n} {c_out}", flush=True)
    w = P(seed=70, n_clouds=1, n=n, radius=0.3, k_cap=5, c_in=9, c_out=c_out)
    rp, ci, v = _pattern(w)
    _assert_tile_forward(n, len(ci), w["M"], 9, c_out)
    t = G.to_device(w)
    csr = G.search(w, t)
    csc = G.sbc.csr_transpose(csr)
    Y = G.sbc.conv_forward(csr, t["F"], t["W"], geometry=G.geometry(w, t))
    assert G.row_error(Y.cpu().numpy(), oracle.conv.forward(rp, ci, v, w["F"], w["W"])) < G.TOL_F32
    # the input gradient of the reversed layer has the same columns
    dF, _ = G.sbc.conv_backward(csr, csc, t["dY"], t["W"].transpose(1, 2).contiguous(), t["F"],
                                geometry=G.geometry(w, t), need_dW=False)
    dF_ref, _ = oracle.conv.backward(rp, ci, v, w["dY"], w["W"].transpose(0, 2, 1), w["F"], n)
    assert G.row_error(dF.cpu().numpy(), dF_ref) < G.TOL_F32
