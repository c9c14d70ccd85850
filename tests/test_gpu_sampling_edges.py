"""The sampler at the sizes where its storage changes (points per thread, the
clouds whose coordinates, rows and neighbours stay on the CU) and the
featureless backward at the edges of its row and column blocks."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from tests import gpu_common as G

pytestmark = pytest.mark.gpu


def _cloud(seed, sizes):
    rng = np.random.default_rng(seed)
    x = np.concatenate([workloads.ellipsoid_surface_points(rng, n, rng.uniform(0.5, 1.0, size=3))
                        for n in sizes if n])
    return x, np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)


# cloud sizes around 4, 8 and 16 points a thread (256 or 512 threads) and the
# 2048 points kept on the CU; the last radius gives more than 24576 edges a cloud
@pytest.mark.parametrize("sizes,radius", [([1024, 1025], 0.08), ([2048], 0.06), ([2049, 64], 0.06),
                                          ([4096, 4097], 0.04), ([900, 3], 0.35)])
@pytest.mark.parametrize("method", ["ifp", "approx_ifp", "approx_ifp_rejection"])
def test_sampling_storage_edges(sizes, radius, method):
    print(f"[sampling edges] {sizes} {method}", flush=True)
    x, splits = _cloud(60 + len(sizes), sizes)
    per = 90
    rp, ci = oracle.points_csr(x, splits, x, splits, radius, 0)
    xd, sd = G.dev(x), G.dev(splits)
    ball = G.sbc.neighbour_search_points(xd, sd, xd, sd, radius, 0)
    if radius == 0.35:
        assert rp[sizes[0]] > 24576
    idx, osp, d2 = G.sbc.sample_points(xd, sd, method, per, ball=ball, with_dmin=True)
    counts = [min(per, n) for n in sizes]
    if method == "ifp":
        ref, dref = oracle.sampling.ifp(x, splits, counts)
    elif method == "approx_ifp":
        ref, dref = oracle.sampling.approx_ifp(x, splits, counts, rp, ci)
    else:
        ref, dref = oracle.sampling.approx_ifp_after_rejection(x, splits, per, rp, ci)
    assert int(osp[-1]) == len(ref)
    assert np.array_equal(idx.cpu().numpy()[:len(ref)], ref)
    assert np.array_equal(d2.cpu().numpy()[:len(x)], dref)


def test_sampling_pattern_without_self_edges():
    """A ball pattern that leaves a point out of its own ball: a taken point is
    still taken once, and its distance is not lowered to 0 by itself."""
    x, splits = _cloud(71, [50])
    rp, ci = oracle.points_csr(x, splits, x, splits, 0.4, 0)
    rows = np.repeat(np.arange(50), np.diff(rp))
    keep = rows != ci
    rp2 = np.concatenate([[0], np.cumsum(np.bincount(rows[keep], minlength=50))]).astype(np.int32)
    ci2 = ci[keep].astype(np.int32)
    ball = G.sbc.CSR(G.dev(rp2), G.dev(ci2), 50, 50, len(ci2))
    idx, _, d2 = G.sbc.sample_points(G.dev(x), G.dev(splits), "approx_ifp", 50, ball=ball,
                                     with_dmin=True)
    ref, dref = oracle.sampling.approx_ifp(x, splits, [50], rp2, ci2)
    assert sorted(idx.cpu().numpy().tolist()) == list(range(50))
    assert np.array_equal(idx.cpu().numpy(), ref) and np.array_equal(d2.cpu().numpy(), dref)


@pytest.mark.parametrize("n,P", [(1, 1), (63, 32), (65, 33), (700, 64), (700, 129)])
@pytest.mark.parametrize("basis", [workloads.BASIS_MONO4, workloads.BASIS_MONO8,
                                   workloads.BASIS_WMONO10])
def test_featureless_block_edges(n, P, basis):
    w = workloads.small_points(seed=72, n_clouds=1, n=n, c_in=1, c_out=P, basis=basis)
    rp, ci = oracle.points_csr(w["x_in"], w["in_splits"], w["x_out"], w["out_splits"], w["radius"],
                               w["k_cap"])
    v = oracle.basis.point_values(basis, w["x_in"], w["x_out"], rp, ci, w["radius"], w["M"])
    t = G.to_device(w)
    csr = G.search(w, t)
    geo = G.geometry(w, t)
    Phi = np.ascontiguousarray(w["W"][:, 0, :])
    Z = G.sbc.featureless_forward(csr, G.dev(Phi), geometry=geo).cpu().numpy()
    dPhi = G.sbc.featureless_backward(csr, t["dY"], w["M"], geometry=geo).cpu().numpy()
    assert G.norm_error(Z, oracle.conv.featureless_forward(rp, ci, v, Phi)[0]) < G.TOL_F32
    assert G.norm_error(dPhi, oracle.conv.featureless_backward(rp, ci, v, w["dY"])) < G.TOL_F32


# batches of more clouds than CUs share them two and three blocks each, with less
# LDS a block for coordinates, rows and neighbours: clouds inside and beyond it
@pytest.mark.parametrize("n_batch", [256, 257, 513])
@pytest.mark.parametrize("method", ["ifp", "approx_ifp", "approx_ifp_rejection", "rejection"])
def test_sampling_many_clouds(n_batch, method):
    print(f"[sampling many] {n_batch} {method}", flush=True)
    sizes = [1 + (7 * i) % 23 for i in range(n_batch)]
    sizes[3], sizes[100], sizes[-1] = 830, 0, 1100
    x, splits = _cloud(90 + n_batch, sizes)
    rp, ci = oracle.points_csr(x, splits, x, splits, 0.2, 0)
    xd, sd = G.dev(x), G.dev(splits)
    ball = G.sbc.neighbour_search_points(xd, sd, xd, sd, 0.2, 0)
    counts = [min(40, n) for n in sizes]
    idx, osp, d2 = G.sbc.sample_points(xd, sd, method, 40, ball=ball, with_dmin=True)
    if method == "ifp":
        ref, dref = oracle.sampling.ifp(x, splits, counts)
    elif method == "approx_ifp":
        ref, dref = oracle.sampling.approx_ifp(x, splits, counts, rp, ci)
    elif method == "approx_ifp_rejection":
        ref, dref = oracle.sampling.approx_ifp_after_rejection(x, splits, 40, rp, ci)
    else:
        taken, dref = oracle.sampling.rejection_sampling(x, splits, rp, ci)
        ref = np.nonzero(taken)[0].astype(np.int32)
    assert int(osp[-1]) == len(ref)
    assert np.array_equal(idx.cpu().numpy()[:len(ref)], ref)
    assert np.array_equal(d2.cpu().numpy()[:len(x)], dref)


# wide dZ: the row sums made once (more than 128 columns), two and four a thread
@pytest.mark.parametrize("n,P", [(64, 128), (65, 256), (63, 257), (1000, 300)])
@pytest.mark.parametrize("basis", [workloads.BASIS_MONO4, workloads.BASIS_WMONO10])
def test_featureless_wide(n, P, basis):
    test_featureless_block_edges(n, P, basis)
