"""Matching with each segment's minima in LDS: exact against the oracle at the
sizes where that path begins and ends, for every policy."""
import numpy as np
import pytest

import oracle
from paper_2012_13618_amd import inputs as I

pytestmark = pytest.mark.gpu


def graph(n, p, dmin, dmax, seed, huge=0):
    """Hyperedges that are runs of consecutive ids (mod n), about p pins in
    all; huge: that many more of 5000 pins."""
    rng = np.random.default_rng(seed)
    d = rng.integers(dmin, dmax + 1, 2 * p // (dmin + dmax))
    d = np.concatenate([d, np.full(huge, 5000)])
    rng.shuffle(d)
    off = np.zeros(len(d) + 1, np.int64)
    np.cumsum(d, out=off[1:])
    start = rng.integers(0, n, len(d))
    pins = (np.repeat(start - off[:-1], d) + np.arange(off[-1])) % n
    return I.Hypergraph(n, off.astype(np.int32), pins.astype(np.int32), np.ones(n, np.int32),
                        rng.integers(1, 9, len(d)).astype(np.int32))


# n at the edges of the rule for few pins, of one range and of the most ranges;
# p at the path's start; empty, wavefront (past a full queue) and workgroup
# hyperedges
@pytest.mark.parametrize("n,p,dmin,dmax,huge", [
    (1, 1 << 18, 1, 1, 0), (40, 1 << 19, 0, 20, 0), (8192, 1 << 18, 2, 12, 0), (8193, 1 << 19, 1, 40, 30),
    (10240, 1 << 19, 33, 90, 100), (10241, 1 << 19, 2, 12, 0), (16384, 1 << 24, 2, 60, 10),
    (16385, 1 << 24, 2, 40, 0), (98304, 1 << 24, 0, 50, 20), (98305, 1 << 24, 20, 50, 0),
])
def test_match(n, p, dmin, dmax, huge):
    import paper_2012_13618_amd as bp
    h = graph(n, p, dmin, dmax, n + p, huge)
    dh = bp.DeviceHypergraph.from_host(h)
    for policy in range(5) if p < 1 << 24 else (bp.LDH, bp.HWD):
        got = bp.step_match(dh, policy).cpu().numpy()
        assert np.array_equal(got, oracle.match(n, h.offsets, h.pins, hw=h.hedge_w, policy=policy)), policy


# runs of hyperedges that span segments: many in one batch, some of one size
@pytest.mark.parametrize("sizes", [[3000] * 64, [9000, 20, 12000, 700, 40, 16000], [200] * 60])
def test_segments(sizes):
    import paper_2012_13618_amd as bp
    hs = [graph(n, max(400, (1 << 19) // len(sizes)), 2, 9, i) for i, n in enumerate(sizes)]
    parts, cuts, _, _ = bp.partition_batch(hs, [2] * len(hs), [0.05] * len(hs))
    for i, h in enumerate(hs):
        ref, cut = oracle.partition(h.num_nodes, h.offsets, h.pins, 2, 0.05, h.node_w, h.hedge_w)
        assert np.array_equal(parts[i], ref) and cuts[i] == cut, i
