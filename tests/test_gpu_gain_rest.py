"""Hyperedges longer than a tile of the hyperedge gain pass: what is counted past the
tile's end, a step of 4096 pins at a time, with whole tiles and quarter ones."""
import numpy as np
import pytest

import oracle
from paper_2012_13618_amd import inputs as I

pytestmark = pytest.mark.gpu


def graph(n, deg, seed=1):
    deg = np.asarray(deg)
    off = np.concatenate([[0], np.cumsum(deg)])
    start = np.random.default_rng(seed).integers(0, n, len(deg))
    # (7919 is prime and no divisor of n: the pins of a hyperedge differ)
    pins = (np.repeat(start, deg) + (np.arange(off[-1]) - np.repeat(off[:-1], deg)) * 7919) % n
    return I.Hypergraph(n, off.astype(np.int32), pins.astype(np.int32), np.ones(n, np.int32),
                        np.random.default_rng(seed + 1).integers(1, 9, len(deg)).astype(np.int32))


@pytest.mark.parametrize("fill", [0, 1100])  # (1100 hyperedges of 4096 pins: whole tiles)
@pytest.mark.parametrize("deg", [1024 + 4095, 1024 + 4096, 1024 + 4097, 8192, 8193, 4096 + 8191, 12289, 40000])
def test_rest(deg, fill):
    import torch
    import paper_2012_13618_amd as bp
    n = 70001
    h = graph(n, [3, deg, 2, deg, deg, 5] + [4096] * fill + [deg + 1])
    for share in (0.0, 0.5, 0.99):
        side = (np.random.default_rng(deg).random(n) < share).astype(np.uint8)
        got = bp.step_gains(bp.DeviceHypergraph.from_host(h), torch.from_numpy(side).cuda()).cpu().numpy()
        assert np.array_equal(got, oracle.gains(n, h.offsets, h.pins, side, h.hedge_w)), share


def test_giant_hyperedge():
    """Half a million pins of one hyperedge against as many in hyperedges of four:
    15 times their time, and 60 times with eight loads a thread and none ahead."""
    import torch
    import paper_2012_13618_amd as bp
    n = 1_000_003
    side = torch.from_numpy((np.random.default_rng(1).random(n) < 0.5).astype(np.uint8)).cuda()
    bp.profile_enable(True)
    try:
        t = []
        for deg in ([500_000], [4] * 125_000):
            h = graph(n, deg)
            off = h.offsets
            h.pins = ((np.arange(off[-1]) - np.repeat(off[:-1], deg)) + np.repeat(h.pins[off[:-1]], deg)).astype(np.int64) % n
            dh = bp.DeviceHypergraph(n, off, h.pins.astype(np.int32), None, None)
            for _ in range(2):
                bp.profile_reset()
                for _ in range(20):
                    bp.step_gains(dh, side)
                t1 = {s["name"]: s["total_ms"] / max(s["launches"], 1) for s in bp.profile_read()}["gain_hedges"]
            t.append(t1)
    finally:
        bp.profile_enable(False)
        bp.profile_reset()
    print(f"one hyperedge {1e3 * t[0]:.1f} us, of four {1e3 * t[1]:.1f}", flush=True)
    assert t[0] < 30 * t[1]
