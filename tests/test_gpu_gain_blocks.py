"""The node pass at the sizes where its form and its number of blocks change - with
the lists' counts and gain extremes, which a swap's selection takes from it - and
that a level of hardly any incidence does not spend its time in their atomics."""
import numpy as np
import pytest

import oracle
from paper_2012_13618_amd import inputs as I

pytestmark = pytest.mark.gpu


# 2^23 pins, at five a node and at 2^18 nodes (staged), 3/4 of 2^20 and an incidence to 16 nodes
# (blocks), 2^15 (blocks of listed nodes; degrees above 32)
@pytest.mark.parametrize("n,pins,d", [
    (1 << 20, 8 << 20, 8), (1 << 20, (8 << 20) - 8, 8), (1677721, 8 << 20, 8), (1677722, 8 << 20, 8), (1 << 18, 8 << 20, 32),
    ((1 << 18) - 1, 8 << 20, 32), (1 << 18, (8 << 20) - 32, 32), (3 << 18, (3 << 18) // 16, 2),
    (3 << 18, (3 << 18) // 16 - 2, 2), ((3 << 18) - 1, 1 << 20, 4), (1 << 15, 40 << 15, 32), ((1 << 15) - 1, 36 << 15, 32),
    (16385, 1 << 19, 64), (513 * 256, 1 << 18, 2), (512 * 256 + 1, 512, 2),
])
def test_swaps(n, pins, d):
    import torch
    import paper_2012_13618_amd as bp
    rng = np.random.default_rng(n)
    e = pins // d
    p = (np.repeat(rng.integers(0, n, e), d) + np.tile(np.arange(d) * 7919, e)) % n
    h = I.Hypergraph(n, np.arange(0, e * d + 1, d, dtype=np.int32), p.astype(np.int32),
                     rng.integers(1, 4, n).astype(np.int32), rng.integers(1, 9, e).astype(np.int32))
    side = (rng.random(n) < 0.45).astype(np.uint8)
    w = int(h.node_w.sum())
    ref, _ = oracle.refine(n, h.offsets, h.pins, side, w, w, 2, h.node_w, h.hedge_w)
    got = torch.from_numpy(side).cuda()
    bp.step_refine(bp.DeviceHypergraph.from_host(h), got, w, w, 2)
    assert np.array_equal(got.cpu().numpy(), ref)


def test_few_incidences_take_few_atomics():
    """Against the pass that flips the chosen nodes, over the same ones: 0.75 of its
    time by 512 blocks, 1.5 by one for every 256 or 512 nodes."""
    import torch
    import paper_2012_13618_amd as bp
    n = 600_003
    rng = np.random.default_rng(1)
    p = np.sort(rng.choice(n, 4000, replace=False)).astype(np.int32)
    dh = bp.DeviceHypergraph(n, torch.arange(0, 4001, 2, dtype=torch.int32).cuda(), torch.from_numpy(p).cuda(), None, None)
    side = torch.from_numpy((rng.random(n) < 0.5).astype(np.uint8)).cuda()
    bp.profile_enable(True)
    try:
        for _ in range(3):
            bp.profile_reset()
            bp.step_refine(dh, side.clone(), n, n, 40)
            got = {s["name"]: s["total_ms"] / max(s["launches"], 1) for s in bp.profile_read()}
    finally:
        bp.profile_enable(False)
        bp.profile_reset()
    print(f"node pass {1e3 * got['gain_nodes']:.1f} us, flips {1e3 * got['flip']:.1f}", flush=True)
    assert got["gain_nodes"] < 1.1 * got["flip"]
