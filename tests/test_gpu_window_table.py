"""The chunk table of the windowed selections: more segments than its workgroup takes
at a time, segments of none, one and several chunks side by side, and its time for
a segment of many chunks."""
import numpy as np
import pytest

import oracle
from paper_2012_13618_amd import inputs as I

pytestmark = pytest.mark.gpu


def windowed(bp):
    s = bp.schedule_default()
    s.fuse_max_pins = 0          # every level by rounds of launches,
    s.seg_select_max_nodes = 0   # and every selection windowed
    bp.schedule_set(s)


@pytest.mark.parametrize("count", [3, 1024, 1025, 2100])
def test_many_segments(count):
    import torch  # (its HIP runtime first)
    torch.cuda.init()
    import paper_2012_13618_amd as bp
    rng = np.random.default_rng(count)
    sizes = rng.integers(1, 40, count)
    sizes[rng.integers(0, count, 6)] = [1023, 1024, 1025, 2048, 2049, 4100]
    sizes[-1] = 3000
    hs = [I.random_small(int(n), max(1, int(n) // 2), 2, 6, i, weighted_nodes=True) for i, n in enumerate(sizes)]
    ks = [2 + i % 3 for i in range(count)]
    old = bp.schedule_get()
    try:
        windowed(bp)
        parts, cuts, _, _ = bp.partition_batch_device([bp.DeviceHypergraph.from_host(h) for h in hs], ks, [0.03] * count)
    finally:
        bp.schedule_set(old)
    for h, k, p, c in zip(hs, ks, parts, cuts):
        ref, cut = oracle.partition_hg(h, k=k, eps=0.03)
        assert np.array_equal(p.cpu().numpy(), ref) and c == cut


def test_time_of_many_chunks():
    """A table of 512 chunks takes about a launch's time (4 launches' by one thread)."""
    import torch
    import paper_2012_13618_amd as bp
    n = 1_000_003
    dh = bp.DeviceHypergraph(n, torch.tensor([0, 2], dtype=torch.int32).cuda(), torch.tensor([0, 1], dtype=torch.int32).cuda(),
                             None, None)
    side = torch.zeros(n, dtype=torch.uint8, device="cuda")
    bp.profile_enable(True)
    try:
        for _ in range(2):
            bp.profile_reset()
            for _ in range(20):
                bp.step_refine(dh, side, n, n, 0)
            got = {s["name"]: s["total_ms"] / max(s["launches"], 1) for s in bp.profile_read()}
    finally:
        bp.profile_enable(False)
        bp.profile_reset()
    print(f"table {1e3 * got['balance']:.1f} us, round test {1e3 * got['round']:.1f}", flush=True)
    assert got["balance"] < 2.5 * got["round"]
