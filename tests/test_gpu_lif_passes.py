"""The spiking sampler where a block's cells take turns in the staging of 2048
entries, at and past the largest cell that fits it, for every number of slots a
pixel reaches, and for the emission's groups of 1024 events."""
import numpy as np
import pytest

import oracle
from tests import gpu_common as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,width,height,kernel,stride", [
    (2048, 1, 1, 1, 1),      # one cell with all the staging
    (2049, 1, 1, 1, 1),      # and one event more
    (4100, 2, 1, 2, 1),      # cells of 2050 and 4100 events
    (1024, 6, 6, 3, 1),      # one group; 9 slots in 3 words
    (1025, 6, 6, 5, 1),      # two groups; 25 slots in 7 words
    (6000, 9, 2, 3, 1),      # a block's cells in several turns, the last partly filled
    (3000, 40, 3, 4, 1),     # 16 slots in 4 words
])
def test_lif_turns(n, width, height, kernel, stride):
    """Cells, times and source events equal the oracle's, in order."""
    print(f"[lif turns] n {n} {width}x{height} k {kernel} s {stride}", flush=True)
    rng = np.random.default_rng(90 + n)
    px = rng.integers(0, width, n).astype(np.int32)
    py = rng.integers(0, height, n).astype(np.int32)
    t = np.sort(rng.integers(0, 20 * n, n)).astype(np.int32)
    ref = oracle.sampling.lif(px, py, t, width, height, kernel, stride, 900.0, 1.3, -1.0)
    x, y, tt, src, cnt = G.sbc.lif_sample_events(G.dev(px), G.dev(py), G.dev(t), width, height,
                                                 kernel, stride, 900.0, 1.3, -1.0)
    assert cnt == len(ref) > 0
    assert np.array_equal(src.cpu().numpy(), ref[:, 0])
    assert np.array_equal(x.cpu().numpy(), ref[:, 1]) and np.array_equal(y.cpu().numpy(), ref[:, 2])
    assert np.array_equal(tt.cpu().numpy(), t[ref[:, 0]])
