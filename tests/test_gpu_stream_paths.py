"""The two paths of a stream batch (linked events up to 8192 of them and 16
rows of G within the LDS, pixel lists beyond) against the oracle's recursion."""
import numpy as np
import pytest

import oracle
import workloads
from tests import gpu_common as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pieces,C_in,P,hot", [
    ([8192], 4, 5, False),       # the largest linked batch
    ([8193], 4, 5, False),       # the smallest one by pixel lists
    ([17, 8193, 15], 3, 17, False),  # both paths on one state
    ([16, 33], 104, 16, False),  # the widest 16 rows of G that fit
    ([16, 33], 112, 16, False),  # and the first that do not
    ([900], 8, 130, True),       # every event on three pixels
])
def test_stream_batch_paths(pieces, C_in, P, hot):
    """Outputs and state within 1e-5 of the recursion (row-normwise: float32
    state and products, other order of the batch sums); times exact."""
    print(f"[stream] pieces {pieces} C_in {C_in} P {P} hot {hot}", flush=True)
    rng = np.random.default_rng(60)
    n, Wd, H, tau = sum(pieces), 18, 14, 3000.0
    px, py, t, _ = workloads.uniform_events(rng, n, Wd, H, 10 * n)
    if hot:
        px, py = np.asarray([3, 4, 4], np.int32)[np.arange(n) % 3], np.full(n, 5, np.int32)
    F = rng.standard_normal((n, C_in)).astype(np.float32)
    W = (rng.standard_normal((8, C_in, P)) / np.sqrt(8 * C_in)).astype(np.float32)
    Y_ref, z_ref, last_ref = oracle.conv.deployment_stream(px, py, t, F.astype(np.float64),
                                                           W.astype(np.float64), Wd, H, tau)
    st = G.sbc.EventStream(Wd, H, C_in, tau, device=G.DEV)
    Ys, a = [], 0
    for k in pieces:
        # features from an odd offset: rows not on 16 bytes
        buf = G.dev(np.concatenate([np.zeros(1, np.float32), F[a:a + k].ravel()]))
        f = buf[1:].view(k, C_in) if len(pieces) > 1 else G.dev(F[a:a + k])
        Ys.append(st.step(G.dev(px[a:a + k]), G.dev(py[a:a + k]), G.dev(t[a:a + k]), f, G.dev(W))
                  .cpu().numpy())
        a += k
    err = G.row_error(np.concatenate(Ys), Y_ref)
    zerr = G.row_error(st.z.cpu().numpy(), z_ref.reshape(-1, C_in))
    print(f"    Y {err:.2e}  z {zerr:.2e}", flush=True)
    assert err < 1e-5 and zerr < 1e-5
    assert np.array_equal(st.z_time.cpu().numpy(), last_ref.reshape(-1).astype(np.int32))


@pytest.mark.parametrize("Mv,C_in,pieces,hot", [
    (1, 3, [8193], False),        # a state per function by pixel lists: longer batches
    (2, 8, [8200, 20], False),    # and one state on both paths
    (4, 27, [40, 300], False),    # the widest 16 rows of G that fit
    (4, 28, [40, 300], False),    # and the first that do not: lists for short batches
    (2, 60, [17, 500], False),
    (4, 8, [700], True),          # every event on three pixels: linked
    (4, 36, [700], True),         # and by lists
])
def test_stream_decays_paths(Mv, C_in, pieces, hot):
    print(f"[stream] Mv {Mv} C_in {C_in} pieces {pieces} hot {hot}", flush=True)
    rng = np.random.default_rng(61)
    n, Wd, H, P = sum(pieces), 18, 14, 20
    px, py, t, _ = workloads.uniform_events(rng, n, Wd, H, 10 * n)
    if hot:
        px, py = np.asarray([3, 4, 4], np.int32)[np.arange(n) % 3], np.full(n, 5, np.int32)
    F = rng.standard_normal((n, C_in)).astype(np.float32)
    W = (rng.standard_normal((8 * Mv, C_in, P)) / np.sqrt(8 * Mv * C_in)).astype(np.float32)
    lam = (rng.uniform(0.5, 2.0, (8, Mv)) / 3000.0).astype(np.float32)
    Y_ref, z_ref, last_ref = oracle.conv.deployment_stream(
        px, py, t, F.astype(np.float64), W.astype(np.float64), Wd, H, None,
        decays=lam.astype(np.float64))
    st = G.sbc.EventStream(Wd, H, C_in, device=G.DEV, decays=G.dev(lam))
    Ys, a = [], 0
    for k in pieces:
        Ys.append(st.step(G.dev(px[a:a + k]), G.dev(py[a:a + k]), G.dev(t[a:a + k]),
                          G.dev(F[a:a + k]), G.dev(W)).cpu().numpy())
        a += k
    assert G.row_error(np.concatenate(Ys), Y_ref) < 1e-5
    assert G.row_error(st.z.cpu().numpy().reshape(-1, C_in), z_ref.reshape(-1, C_in)) < 1e-5
    assert np.array_equal(st.z_time.cpu().numpy().ravel(),
                          last_ref.reshape(-1).astype(np.int32))
