"""The incidence of small levels by one workgroup: at the sizes where that path
ends (nodes and half the pins 36864, or 16384 hyperedges), with more large hyperedges than
its queue holds and with nodes of every bucket; exact against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2012_13618_amd import inputs as I

pytestmark = pytest.mark.gpu


def graph(n, degs, hubs, seed):
    """Runs of consecutive ids (mod n); hub i is added to the next `count` hyperedges that lack it."""
    rng = np.random.default_rng(seed)
    lists = [set(((s + np.arange(d)) % n).tolist()) for s, d in zip(rng.integers(0, n, len(degs)), degs)]
    for v, count in hubs:
        for x in lists:
            if count > 0 and v not in x:
                x.add(v)
                count -= 1
    off = np.concatenate([[0], np.cumsum([len(x) for x in lists])])
    pins = np.array([v for x in lists for v in sorted(x)], np.int32)
    return I.Hypergraph(n, off.astype(np.int32), pins, rng.integers(1, 4, n).astype(np.int32),
                        rng.integers(1, 4, len(lists)).astype(np.int32))


@pytest.mark.parametrize("n,degs,hubs", [
    (1, [1], []), (50, [], []), (4096, [4] * 16384, []), (4096, [4] * 16383 + [5], []), (4097, [4] * 16383 + [3], []),
    (30000, [2] * 6864, []), (30000, [2] * 6863 + [3], []), (36864, [], []),
    (3000, [2] * 16385, []), (3000, [2] * 16384, [(5, 33), (6, 32), (7, 2048), (8, 2049), (2999, 16000)]),
    (700, [33] * 1500, [(0, 1500)]), (9000, [4500, 300, 65, 64, 33, 32, 0, 1] * 12, []),
    (1025, [7] * 2040, [(1, 2040)]), (1024, [7] * 2060, [(1, 2060)]),
])
def test_small_levels(n, degs, hubs):
    import torch
    import paper_2012_13618_amd as bp
    h = graph(n, degs, hubs, n + len(degs))
    dh = bp.DeviceHypergraph.from_host(h)
    for policy in (bp.LDH, bp.HWD):
        got = bp.step_match(dh, policy).cpu().numpy()
        assert np.array_equal(got, oracle.match(n, h.offsets, h.pins, hw=h.hedge_w, policy=policy))
    side = (np.random.default_rng(1).random(n) < 0.4).astype(np.uint8)
    got = bp.step_gains(dh, torch.from_numpy(side).cuda()).cpu().numpy()
    assert np.array_equal(got, oracle.gains(n, h.offsets, h.pins, side, h.hedge_w))
    part, cut, _, _ = bp.partition_device(dh, 3, 0.1)
    ref, rcut = oracle.partition(n, h.offsets, h.pins, 3, 0.1, h.node_w, h.hedge_w)
    assert np.array_equal(part.cpu().numpy(), ref) and cut == rcut
