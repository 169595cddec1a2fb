"""Coarse levels of small segments in one launch (and the one-workgroup rounds
they share) against the oracle: more levels than one launch takes, the limits of
nodes and pins, hyperedges a thread, 16 lanes or a wavefront take, more of them
than the queue holds, every number of swaps, uneven parts."""
import numpy as np
import pytest

import oracle
from paper_2012_13618_amd import inputs as I

pytestmark = pytest.mark.gpu


def check(h, k=2, eps=0.05, **prm):
    import paper_2012_13618_amd as bp
    part, cut, _, rep = bp.partition_device(bp.DeviceHypergraph.from_host(h), k, eps, bp.params(**prm))
    want, want_cut = oracle.partition(h.num_nodes, h.offsets, h.pins, k, eps, h.node_w, h.hedge_w,
                                      oracle.params(**prm))
    assert np.array_equal(part.cpu().numpy(), want) and cut == want_cut
    return rep


def pairs(n, seed):
    """A path over n nodes in random order: every level halves it."""
    v = np.random.default_rng(seed).permutation(n).astype(np.int32)
    pins = np.sort(np.stack([v[:-1], v[1:]], 1), axis=1).reshape(-1)
    return I.Hypergraph(n, np.arange(0, 2 * n - 1, 2, dtype=np.int32), pins.astype(np.int32), np.ones(n, np.int32),
                        np.ones(n - 1, np.int32))


@pytest.mark.parametrize("iters", [0, 1, 2, 3])
def test_many_levels(iters):
    rep = check(pairs(6000, 3), k=3, refine_iters=iters, min_coarse_nodes=0)
    assert rep.coarsen_levels > 9  # more than one launch


@pytest.mark.parametrize("n,e,dmin,dmax", [
    (8192, 9000, 2, 4), (8193, 9000, 2, 4), (300, 3000, 15, 18), (400, 1000, 60, 70), (2000, 6000, 2, 20),
    (600, 5900, 10, 12), (50, 900, 2, 40), (2, 1, 2, 2), (3, 0, 2, 2),
])
@pytest.mark.parametrize("weighted", [False, True])
def test_limits(n, e, dmin, dmax, weighted):
    h = I.random_small(n, e, dmin, min(dmax, n), n + e, weighted_nodes=weighted, weighted_hedges=weighted)
    check(h, k=2)
    check(h, k=5, eps=0.02, min_coarse_nodes=7)


def test_queue_overflow():
    # 7000 hyperedges of 17 or 18 pins in one segment of 120 K pins (queue: 4096)
    import torch
    import paper_2012_13618_amd as bp
    h = I.random_small(900, 7000, 17, 18, 5)
    for frac in (0.9, 0.3):
        side = (np.random.default_rng(1).random(900) < frac).astype(np.uint8)
        ref, stuck = oracle.refine(900, h.offsets, h.pins, side, 460, 460, iters=1, nw=h.node_w, hw=h.hedge_w)
        got = torch.as_tensor(side.copy()).cuda()
        assert bp.step_refine(bp.DeviceHypergraph.from_host(h), got, 460, 460, iters=1) == stuck
        assert np.array_equal(got.cpu().numpy(), ref)
