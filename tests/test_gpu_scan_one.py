"""Prefix scans at the sizes where one workgroup ends (2048 and 8192 elements):
nodes and hyperedges of a level, exact against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2012_13618_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 1023, 2047, 2048, 2049, 8191, 8192, 8193])
@pytest.mark.parametrize("e", [1, 2048, 2049, 8192, 8193])
def test_sizes(n, e):
    import paper_2012_13618_amd as bp
    rng = np.random.default_rng(n + e)
    deg = np.minimum(rng.integers(0, 7, e), n)
    off = np.concatenate([[0], np.cumsum(deg)])
    start = rng.integers(0, n, e)
    pins = (np.repeat(start - off[:-1], deg) + np.arange(off[-1])) % n
    h = I.Hypergraph(n, off.astype(np.int32), pins.astype(np.int32), rng.integers(1, 4, n).astype(np.int32),
                     rng.integers(1, 4, e).astype(np.int32))
    dh = bp.DeviceHypergraph.from_host(h)
    got = [t.cpu().numpy() for t in bp.step_coarsen(dh)]
    for what, a, b in zip(["parent", "offsets", "pins", "node_w", "hedge_w"], got,
                          oracle.coarsen(n, h.offsets, h.pins, h.node_w, h.hedge_w)):
        assert np.array_equal(a, b), what
    part, cut, _, _ = bp.partition_device(dh, 3, 0.1)
    ref, rcut = oracle.partition(n, h.offsets, h.pins, 3, 0.1, h.node_w, h.hedge_w)
    assert np.array_equal(part.cpu().numpy(), ref) and cut == rcut
