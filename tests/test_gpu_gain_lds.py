"""Gains with each segment's gains in LDS: exact against the oracle at the sizes
where that path begins and ends, and through the refinement that uses it."""
import numpy as np
import pytest

import oracle
from paper_2012_13618_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bp():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2012_13618_amd as mod
    mod.lib()
    return mod


def runs_graph(n, p, dmin, dmax, seed, max_w=1, huge=0):
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
                        rng.integers(1, max_w + 1, len(d)).astype(np.int32))


# n at the edges of the two LDS sizes and one past the larger (the passes
# again); p at the path's start; 1-pin and empty hyperedges, wavefront ones
# with a full queue, workgroup ones, weights past the packed contributions
@pytest.mark.parametrize("n,p,dmin,dmax,max_w,huge", [
    (1, 1 << 20, 1, 1, 3, 0), (63, 1 << 20, 0, 20, 3, 0), (16384, 1 << 20, 1, 40, 3, 0),
    (16385, 16385 * 64 + 100, 2, 33, 70000, 20), (36864, 36864 * 64 + 100, 2, 90, 3, 100),
    (36865, 36865 * 64 + 100, 2, 90, 3, 10), (5000, 1 << 20, 2, 4, 1, 300), (40, 20_000_000, 33, 40, 2, 0),
])
def test_gains(bp, n, p, dmin, dmax, max_w, huge):
    import torch
    h = runs_graph(n, p, dmin, dmax, n + p, max_w, huge)
    dh = bp.DeviceHypergraph.from_host(h)
    for share in (0.0, 0.3, 1.0):
        side = (np.random.default_rng(7).random(n) < share).astype(np.uint8)
        got = bp.step_gains(dh, torch.from_numpy(side).cuda()).cpu().numpy()
        assert np.array_equal(got, oracle.gains(n, h.offsets, h.pins, side, h.hedge_w)), share


# swaps (whole lists on both sides) and balance rounds whose gains start here
# and are updated from the moves
@pytest.mark.parametrize("n,p,dmax", [(3000, 1 << 20, 30), (16384, 1 << 20, 12), (20000, 20000 * 64 + 100, 50)])
def test_refine(bp, n, p, dmax):
    import torch
    h = runs_graph(n, p, 2, dmax, n, 3)
    dh = bp.DeviceHypergraph.from_host(h)
    side = (np.random.default_rng(3).random(n) < 0.35).astype(np.uint8)
    lim = int(n * 0.52)
    want = np.asarray(oracle.refine(n, h.offsets, h.pins, side.copy(), lim, lim, 2, h.node_w, h.hedge_w)[0])
    got = torch.from_numpy(side.copy()).cuda()
    bp.step_refine(dh, got, lim, lim, 2)
    assert np.array_equal(got.cpu().numpy(), want)
