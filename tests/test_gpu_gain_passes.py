"""The hyperedge and node passes of the gains against the oracle: hyperedges that
end at, before and past a tile of 4096 pins, node degrees around the staged
limit of 64 and the big nodes', both forms of the contributions, and the levels
large enough for side and contribution bits."""
import numpy as np
import pytest

import oracle
from paper_2012_13618_amd import inputs as I

pytestmark = pytest.mark.gpu
T = 4096


def check(h, seed=0):
    import torch
    import paper_2012_13618_amd as bp
    dh = bp.DeviceHypergraph.from_host(h)
    for share in (0.0, 0.4, 0.999):
        side = (np.random.default_rng(seed).random(h.num_nodes) < share).astype(np.uint8)
        got = bp.step_gains(dh, torch.from_numpy(side).cuda()).cpu().numpy()
        assert np.array_equal(got, oracle.gains(h.num_nodes, h.offsets, h.pins, side, h.hedge_w)), share


def graph(n, deg, max_w, seed=1):
    rng = np.random.default_rng(seed)
    off = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    start = rng.integers(0, n, len(deg))
    pins = (np.repeat(start - off[:-1], deg) + np.arange(off[-1])) % n
    return I.Hypergraph(n, off, pins.astype(np.int32), np.ones(n, np.int32),
                        rng.integers(1, max_w + 1, len(deg)).astype(np.int32))


@pytest.mark.parametrize("max_w", [1, 70000])
@pytest.mark.parametrize("deg", [
    [2], [T], [T - 1, 2], [T - 1, 1, 1], [T, T, 5], [3, 3 * T + 9, 4], [2] * (T // 2) + [3], [1, 0, 0, T + 1, 0, 7, 0], [T, 0, T, 0, 0], [0, 2 * T, 0, 0],
    [64] * 200, [65] * 200, [T // 2 + 1] * 7, list(range(90)),
], ids=str)
def test_tiles(deg, max_w):
    check(graph(40000, np.array(deg), max_w))


# every node in exactly r hyperedges of two pins: the staged limit, the listed
# nodes and (a hub) the big ones
@pytest.mark.parametrize("r", [1, 15, 16, 17, 63, 64, 65, 130])
def test_node_degrees(r):
    n = 1000
    v = np.arange(n)
    pins = np.stack([np.concatenate([v] * ((r + 1) // 2)),
                     np.concatenate([(v + 1 + k) % n for k in range((r + 1) // 2)])], 1)
    hub = np.stack([np.full(9000, n), np.random.default_rng(r).integers(0, n, 9000)], 1)
    pins = np.concatenate([pins, hub]).astype(np.int32)
    e = len(pins)
    check(I.Hypergraph(n + 1, np.arange(0, 2 * e + 1, 2, dtype=np.int32), pins.reshape(-1),
                       np.ones(n + 1, np.int32), np.random.default_rng(r).integers(1, 9, e).astype(np.int32)))


@pytest.mark.parametrize("n,e", [(2 << 20, 500_000), ((2 << 20) - 1, (1 << 20) + 1), (50_000, 1 << 20)])
def test_bits_of_large_levels(n, e):
    h = I.uniform_hypergraph(n, e, 2, 5, n % 1000)
    check(h)
