"""Coarse hyperedge lists at the sizes where the way they are built changes (8, 16,
32, 64, 256, 512, 1024 and 8192 pins), with many pins of one parent and none:
exact against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2012_13618_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [2, 7, 8, 9, 15, 16, 17, 31, 32, 33, 63, 64, 65, 255, 256, 257, 512, 513, 1024, 1025,
                               8192, 8193])
@pytest.mark.parametrize("n", [9000, 40000])
def test_sizes(d, n):
    import paper_2012_13618_amd as bp
    rng = np.random.default_rng(d + n)
    # hyperedges of d - 1, d and d + 1 pins among many pairs, which decide the groups
    deg = np.concatenate([rng.integers(max(2, d - 1), d + 2, 70 if d < 300 else 5), np.full(n // 2, 2)])
    rng.shuffle(deg)
    pins = np.concatenate([np.sort(rng.choice(n, k, replace=False)) for k in deg])
    off = np.concatenate([[0], np.cumsum(deg)])
    h = I.Hypergraph(n, off.astype(np.int32), pins.astype(np.int32), np.ones(n, np.int32),
                     np.ones(len(deg), np.int32))
    got = [t.cpu().numpy() for t in bp.step_coarsen(bp.DeviceHypergraph.from_host(h))]
    ref = oracle.coarsen(n, h.offsets, h.pins, h.node_w, h.hedge_w)
    for what, a, b in zip(["parent", "offsets", "pins", "node_w", "hedge_w"], got, ref):
        assert np.array_equal(a, b), what
