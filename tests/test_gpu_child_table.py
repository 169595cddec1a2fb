"""Children of a tree level with more sides than the table's workgroup has
threads, and at its edge, some of them done: exact against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2012_13618_amd import inputs as I

pytestmark = pytest.mark.gpu


def graph(n, seed):
    rng = np.random.default_rng(seed)
    deg = rng.integers(2, 6, 2 * n)
    off = np.concatenate([[0], np.cumsum(deg)])
    pins = np.concatenate([np.sort(rng.choice(n, d, replace=False)) for d in deg])
    return I.Hypergraph(n, off.astype(np.int32), pins.astype(np.int32), rng.integers(1, 4, n).astype(np.int32),
                        rng.integers(1, 4, len(deg)).astype(np.int32))


@pytest.mark.parametrize("k", [1, 2, 3, 511, 512, 513, 1025])
def test_many_parts(k):
    import paper_2012_13618_amd as bp
    h = graph(6000, k)
    part, cut, _, _ = bp.partition_device(bp.DeviceHypergraph.from_host(h), k, 0.1)
    ref, rcut = oracle.partition(h.num_nodes, h.offsets, h.pins, k, 0.1, h.node_w, h.hedge_w)
    assert np.array_equal(part.cpu().numpy(), ref) and cut == rcut


@pytest.mark.parametrize("n", [255, 256, 257, 600])
def test_many_members(n):
    import paper_2012_13618_amd as bp
    hs = [graph(30 + i % 40, i) for i in range(n)]
    ks = [2 + i % 4 for i in range(n)]
    parts, cuts, _, _ = bp.partition_batch(hs, ks, [0.1] * n)
    for i, h in enumerate(hs):
        ref, rcut = oracle.partition(h.num_nodes, h.offsets, h.pins, ks[i], 0.1, h.node_w, h.hedge_w)
        assert np.array_equal(parts[i], ref) and cuts[i] == rcut, i
