"""Balance rounds whose gains follow the moves: hyperedges at the sizes where a
thread, a wavefront or the workgroup spreads a change, counts of one and two on
a side, weights past the packed contributions, nodes moved that share most of
their hyperedges."""
import numpy as np
import pytest

import oracle
from paper_2012_13618_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dmin,dmax,e", [(1, 3, 9000), (8, 9, 4000), (31, 34, 2000), (2047, 2049, 60), (2, 40, 5000)])
@pytest.mark.parametrize("max_w", [1, 40000])
def test_rounds(dmin, dmax, e, max_w):
    import torch
    import paper_2012_13618_amd as bp
    n = 6000
    h = I.random_small(n, e, dmin, dmax, dmax + max_w, weighted_nodes=True)
    h.hedge_w = np.random.default_rng(e).integers(1, max_w + 1, e).astype(np.int32)
    total = int(h.node_w.sum())
    old = bp.schedule_get()
    try:
        s = bp.schedule_default()
        s.fuse_max_pins, s.incremental_min_pins = 0, 0
        bp.schedule_set(s)
        dh = bp.DeviceHypergraph.from_host(h)
        # all on one side (every hyperedge becomes cut as its first pin moves), then scattered
        for side in (np.ones(n, np.uint8), (np.random.default_rng(3).random(n) < 0.2).astype(np.uint8)):
            lim = total * 51 // 100
            ref, stuck = oracle.refine(n, h.offsets, h.pins, side, lim, lim, iters=0, nw=h.node_w, hw=h.hedge_w)
            got = torch.as_tensor(side.copy()).cuda()
            assert bp.step_refine(dh, got, lim, lim, iters=0) == stuck
            assert np.array_equal(got.cpu().numpy(), ref)
    finally:
        bp.schedule_set(old)
