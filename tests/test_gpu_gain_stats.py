"""Selections by the lists' sizes and gain extremes that the node pass records, on
levels too large for one workgroup and too small for the staged pass: most nodes
have no hyperedge, so three wavefronts of four reach the records at once while
the one that clears them has the nodes with hyperedges."""
import numpy as np
import pytest

import oracle
from paper_2012_13618_amd import inputs as I

pytestmark = pytest.mark.gpu


def graph(n, seed):
    rng = np.random.default_rng(seed)
    v = np.arange(n)
    v = v[v % 256 < 64]  # the nodes of each workgroup's first wavefront
    pairs = np.stack([np.tile(v, 3), rng.permutation(np.tile(v, 3))], 1)
    pairs = pairs[pairs[:, 0] != pairs[:, 1]].astype(np.int32)
    e = len(pairs)
    return I.Hypergraph(n, np.arange(0, 2 * e + 1, 2, dtype=np.int32), pairs.reshape(-1),
                        rng.integers(1, 4, n).astype(np.int32), rng.integers(1, 9, e).astype(np.int32))


@pytest.mark.parametrize("n", [16385, 40000, 133000, (1 << 18) - 1])
def test_refine_and_initial(n):
    import torch
    import paper_2012_13618_amd as bp
    h = graph(n, n)
    dh = bp.DeviceHypergraph.from_host(h)
    w = int(h.node_w.sum())
    for share in (0.5, 0.1, 0.97):
        side = (np.random.default_rng(n + 1).random(n) < share).astype(np.uint8)
        ref, stuck = oracle.refine(n, h.offsets, h.pins, side, w // 2 + 10, w // 2 + 10, 2, h.node_w, h.hedge_w)
        got = torch.from_numpy(side).cuda()
        assert bp.step_refine(dh, got, w // 2 + 10, w // 2 + 10, 2) == stuck, share
        assert np.array_equal(got.cpu().numpy(), ref), share
    ref = oracle.initial(n, h.offsets, h.pins, 2, 1, h.node_w, h.hedge_w)
    assert np.array_equal(bp.step_initial(dh, 2, 1).cpu().numpy(), ref)
