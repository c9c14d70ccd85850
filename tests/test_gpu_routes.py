"""The choice between the tile passes and the separate kernels: shapes at which
each is taken (the launches say which ran), in both directions, against the
oracle, under AUTO and with the basis values given; rows of very different
lengths; the forward whose space is fixed."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import workloads
from paper_2012_01170_amd import _lib
from tests import gpu_common as G

pytestmark = pytest.mark.gpu

P, E = workloads.small_points, workloads.small_events
M4, M8, W10 = workloads.BASIS_MONO4, workloads.BASIS_MONO8, workloads.BASIS_WMONO10


def _sparse(seed, n, c_in, c_out, basis=M8, dtype="f32", radius=0.04):
    """Short rows: about three entries."""
    return P(seed=seed, n_clouds=2, n=n // 2, radius=radius, c_in=c_in, c_out=c_out, basis=basis,
             dtype=dtype)


def _events(seed, n, c, n_decays, dtype="f32"):
    """Short rows: about two entries."""
    return E(seed=seed, n=n, width=64, height=64, duration_us=100_000, window_us=int(9e7 / n),
             c=c, n_decays=n_decays, dtype=dtype)


def _crowded(seed, basis, c_in, c_out):
    """A few rows of 130 entries among short ones."""
    rng = workloads.rng_for(6, salt=seed + 1)
    a = workloads.ellipsoid_surface_points(rng, 130, np.full(3, 0.01))
    b = workloads.ellipsoid_surface_points(rng, 6000, np.full(3, 1.0))
    return workloads.points_workload(rng, [(a, a), (b, b)], basis, 0.03, 0, c_in, c_out)


# name -> workload, forward and backward on the tile passes
ROUTES = {
    "mono4_wide_in": (lambda: _sparse(80, 1500, 130, 65, M4, radius=0.06), True, True),
    "wide_out": (lambda: _sparse(81, 17000, 32, 129, radius=0.02), True, True),
    "weighted": (lambda: _sparse(82, 9000, 40, 72, W10, radius=0.025), True, True),
    "bf16_wide": (lambda: _sparse(83, 5000, 64, 132, M4, "bf16"), True, True),
    "bf16_weighted": (lambda: _sparse(84, 6000, 36, 68, W10, "bf16"), True, True),
    "crowded": (lambda: _crowded(85, M8, 20, 36), True, True),
    "crowded_weighted": (lambda: _crowded(86, W10, 16, 16), True, True),
    "decays3": (lambda: _events(87, 40000, 24, 3), True, True),
    "decays3_bf16": (lambda: _events(88, 40000, 32, 3, "bf16"), True, True),
    "decays4": (lambda: _events(89, 40000, 32, 4), True, True),
    # the separate kernels: long rows of many basis functions, wide channels
    "long_rows": (lambda: P(seed=90, n_clouds=2, n=200, radius=3.0, k_cap=0, c_in=20, c_out=36),
                  False, False),
    "narrowing": (lambda: P(seed=91, c_in=256, c_out=8), False, True),
    "widening": (lambda: P(seed=92, c_in=8, c_out=256), True, False),
    "square_wide": (lambda: P(seed=93, c_in=128, c_out=128), True, False),
    "narrowing_bf16": (lambda: P(seed=94, c_in=200, c_out=16, dtype="bf16"), False, True),
    "narrowing_weighted": (lambda: P(seed=95, c_in=300, c_out=9, basis=W10, n_out=40), False, True),
    "square_wider": (lambda: P(seed=97, c_in=256, c_out=256), False, False),
    "decays4_small": (lambda: E(seed=96, n=1100, c=9, n_decays=4), True, False),
    "decays4_long": (lambda: E(seed=98, n=1500, c=12, n_decays=4, window_us=15_000), False, False),
}
TILE = ("fwd_fused", "bwd_tile_df", "bwd_tile_dw")


def _ran(names, f):
    """f(), and which of the traced launches it made."""
    L = _lib.lib()
    pairs = {}
    for k in names:
        # (a recorded event's time changes; each pair starts with one far apart)
        pairs[k] = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        for e in pairs[k]:
            e.record()
    torch.cuda.synchronize()
    mark = torch.cuda.Event(enable_timing=True)
    mark.record()
    mark.synchronize()
    for k, (a, b) in pairs.items():
        _lib.check(L.sbc_trace_kernel(k.encode(), ctypes.c_void_p(a.cuda_event),
                                      ctypes.c_void_p(b.cuda_event)))
    try:
        out = f()
    finally:
        L.sbc_trace_clear()
    torch.cuda.synchronize()
    return out, {k for k, (a, b) in pairs.items() if mark.elapsed_time(b) > 0}


def _pattern(w):
    if w["kind"] == "points":
        rp, ci = oracle.points_csr(w["x_in"], w["in_splits"], w["x_out"], w["out_splits"],
                                   w["radius"], w["k_cap"])
        return rp, ci, oracle.basis.point_values(w["basis"], w["x_in"], w["x_out"], rp, ci,
                                                 w["radius"], w["M"])
    rp, ci = oracle.events_csr(w["px"], w["py"], w["t"], w["window"], 1, w["width"], w["height"])
    return rp, ci, oracle.basis.event_values(w["basis"], w["px"], w["py"], w["t"], rp, ci,
                                             w["tau"], w.get("decays"))


@pytest.mark.parametrize("name", list(ROUTES))
def test_routes(name):
    print(f"[routes] {name}", flush=True)
    make, fwd_tile, bwd_tile = ROUTES[name]
    w = make()
    rp, ci, v = _pattern(w)
    t = G.to_device(w)
    csr = G.search(w, t)
    csc = G.sbc.csr_transpose(csr)
    geo = G.geometry(w, t)
    Y_ref = oracle.conv.forward(rp, ci, v, w["F"], w["W"])
    dF_ref, dW_ref = oracle.conv.backward(rp, ci, v, w["F"], w["W"], w["dY"], w["n_in"])
    vd = torch.from_numpy(np.ascontiguousarray(v, dtype=np.float32)).to(G.DEV)
    for given in (False, True):
        kw = dict(v=vd) if given else dict(geometry=geo)
        (Y, (dF, dW)), ran = _ran(TILE, lambda: (
            G.sbc.conv_forward(csr, t["F"], t["W"], **kw),
            G.sbc.conv_backward(csr, csc, t["F"], t["W"], t["dY"], **kw)))
        if not given:
            assert ("fwd_fused" in ran) == fwd_tile
            assert {"bwd_tile_df", "bwd_tile_dw"} & ran == (set(TILE[1:]) if bwd_tile else set())
        assert G.row_error(Y.cpu().numpy(), Y_ref) < G.TOL_F32
        assert G.row_error(dF.cpu().numpy(), dF_ref) < G.TOL_F32
        assert G.norm_error(dW.cpu().numpy(), dW_ref) < G.TOL_F32


def test_fixed_space_takes_the_tile_pass():
    """Where the separate kernels' intermediate does not fit the library's
    scratch, the forward without a workspace gathers and contracts in one pass."""
    n, M, ci, co = 20000, 8, 512, 8
    k = 24
    gen = torch.Generator(device=G.DEV)
    gen.manual_seed(6)
    rp = torch.arange(0, n * k + 1, k, dtype=torch.int32, device=G.DEV)
    idx = torch.randint(0, n, (n * k,), generator=gen, device=G.DEV, dtype=torch.int32)
    csr = G.sbc.CSR(rp, idx, n, n, n * k)
    v = torch.rand((n * k, M), generator=gen, device=G.DEV)
    F = torch.randn((n, ci), generator=gen, device=G.DEV)
    W = torch.randn((M, ci, co), generator=gen, device=G.DEV)
    ref = G.sbc.conv_forward(csr, F, W, v=v, order="gemm_first").double().cpu().numpy()
    Y = torch.empty((n, co), device=G.DEV)
    _, ran = _ran(("fwd_fused",), lambda: G.sbc.conv_forward_noalloc(csr, F, W, Y, v=v,
                                                                     order="spmm_first"))
    assert ran == {"fwd_fused"}
    assert G.row_error(Y.cpu().numpy(), ref) < G.TOL_F32
