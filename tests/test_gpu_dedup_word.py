"""Hyperedges with different pins whose fingerprints agree in the bits that the
duplicate table keeps and in their slot: told apart, merged only with their own
duplicates, exact against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2012_13618_amd import inputs as I

pytestmark = pytest.mark.gpu

NC = 8192                       # coarse nodes, each a pair of nodes
SETS = [(984, 1397), (1393, 4663)]  # two coarse pairs, found by search


def mix(z):
    with np.errstate(over="ignore"):
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
    return z ^ (z >> np.uint64(31))


@pytest.mark.parametrize("order", [[0, 1], [1, 0], [0, 1, 0, 1], [1, 1, 0, 0, 1], [0] * 3 + [1] * 70 + [0] * 70])
@pytest.mark.parametrize("apart", [0, 100])
def test_shared_bits(order, apart):
    import paper_2012_13618_amd as bp
    t = mix(np.arange(NC, dtype=np.uint64))
    with np.errstate(over="ignore"):
        f = [t[a] + t[b] + np.uint64(2) * np.uint64(0x9E3779B97F4A7C15) for a, b in SETS]
    assert f[0] != f[1] and f[0] >> np.uint64(31) == f[1] >> np.uint64(31)
    assert len({int((x ^ (x >> np.uint64(32))) & np.uint64(32767)) for x in f}) == 1  # the table's 2^15 slots

    # a pair of nodes per coarse node, then the sets as triples (a larger degree: never first)
    edges = [[2 * i, 2 * i + 1] for i in range(NC)]
    for k, s in enumerate(order):
        a, b = SETS[s]
        edges.append(sorted([2 * a, 2 * a + 1, 2 * b]))
        edges += [[2 * j, 2 * j + 1, 2 * j + 2] for j in range(6000 + 2, 6000 + 2 + apart // len(order))]
    E = len(edges)
    assert 8192 < E <= 16384
    deg = np.array([len(e) for e in edges])
    off = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    h = I.Hypergraph(2 * NC, off, np.concatenate(edges).astype(np.int32), np.ones(2 * NC, np.int32),
                     np.arange(1, E + 1).astype(np.int32) % 7 + 1)
    got = [x.cpu().numpy() for x in bp.step_coarsen(bp.DeviceHypergraph.from_host(h))]
    ref = oracle.coarsen(2 * NC, h.offsets, h.pins, h.node_w, h.hedge_w)
    assert np.array_equal(ref[0][:20:2], np.arange(10))
    for what, a, b in zip(["parent", "offsets", "pins", "node_w", "hedge_w"], got, ref):
        assert np.array_equal(a, b), what
