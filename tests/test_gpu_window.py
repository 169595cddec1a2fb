"""The windowed balance selection against the oracle: chunk and tile edges, gains
far wider than the window and far outside it, nodes of many incidences moved,
zero weights, the whole list moved, no move possible."""
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
    old = mod.schedule_get()
    s = mod.schedule_default()
    s.fuse_max_pins = 0          # every level by rounds of launches,
    s.seg_select_max_nodes = 0   # and every selection windowed
    s.incremental_min_pins = 0
    mod.schedule_set(s)
    yield mod
    mod.schedule_set(old)


def check(bp, h, side, m0, m1, iters=0):
    import torch
    n = h.num_nodes
    ref, stuck = oracle.refine(n, h.offsets, h.pins, side, m0, m1, iters=iters, nw=h.node_w, hw=h.hedge_w)
    got = torch.as_tensor(side.copy()).cuda()
    gs = bp.step_refine(bp.DeviceHypergraph.from_host(h), got, m0, m1, iters=iters)
    assert np.array_equal(got.cpu().numpy(), ref) and gs == stuck


@pytest.mark.parametrize("n", [1, 2, 63, 255, 1023, 1024, 1025, 2047, 2048, 2049, 4097, 50000])
@pytest.mark.parametrize("max_w", [1, 5, 400, 200000])
def test_sizes_and_spans(bp, n, max_w):
    rng = np.random.default_rng(n + max_w)
    h = I.random_small(n, max(1, n), 2, 9, n + 3, weighted_nodes=n % 2 == 0)
    e = h.num_hedges
    h.hedge_w = rng.integers(1, max_w + 1, e).astype(np.int32)
    if max_w > 1000:  # a few far outliers above and below
        h.hedge_w[rng.integers(0, e, min(e, 3))] = 3_000_000
    total = int(h.node_w.sum())
    for frac in (0.9, 0.2):
        side = (rng.random(n) < frac).astype(np.uint8)
        check(bp, h, side, int(total * 0.55), int(total * 0.55))


def test_all_gains_above_the_first_window(bp):
    # one side's nodes each alone in a heavy hyperedge: gains of tens of thousands
    n = 5000
    pairs = np.arange(n, dtype=np.int32)
    h = I.Hypergraph(n, np.arange(0, n + 1, 2, dtype=np.int32), pairs, np.ones(n, np.int32),
                     np.random.default_rng(1).integers(20000, 90000, n // 2).astype(np.int32))
    side = (pairs % 2 == 0).astype(np.uint8)
    side[: n // 4] = 1
    check(bp, h, side, n * 52 // 100, n * 52 // 100)
    # and below it: no hyperedge cut
    check(bp, h, np.ones(n, np.uint8), n * 52 // 100, n * 52 // 100)


def test_hubs_zero_weights_and_stuck(bp):
    rng = np.random.default_rng(9)
    n, e = 3000, 40000
    # 100 hubs in most hyperedges
    pins = np.stack([rng.integers(0, 100, e), rng.integers(100, 1500, e), rng.integers(1500, n, e)], 1)
    h = I.Hypergraph(n, np.arange(0, 3 * e + 1, 3, dtype=np.int32), pins.reshape(-1).astype(np.int32),
                     np.ones(n, np.int32), np.ones(e, np.int32))
    check(bp, h, np.ones(n, np.uint8), n // 2, n // 2)
    h.node_w = (rng.random(n) < 0.5).astype(np.int32)
    w = int(h.node_w.sum())
    check(bp, h, np.ones(n, np.uint8), w // 2, w // 2 + 1)
    # all of the heavy side's nodes wanted, and none fits the other side
    h.node_w = np.full(n, 7, np.int32)
    side = np.zeros(n, np.uint8)
    side[:40] = 1
    check(bp, h, side, 7 * n, 0)
    check(bp, h, side, 7 * (n - 40) + 3, 100)


def test_large_segment(bp):
    n = 1_200_000  # chunks of more than one tile
    h = I.uniform_hypergraph(n, n // 4, 2, 5, 11)
    side = (np.random.default_rng(2).random(n) < 0.54).astype(np.uint8)
    check(bp, h, side, n * 53 // 100, n * 53 // 100)
