"""The autotuner runs no two schedules that select in the same way (one-workgroup
selections end at 16384 nodes whatever larger limit is set)."""
import pytest

from paper_2012_13618_amd import inputs as I

pytestmark = pytest.mark.gpu


def test_one_run_a_schedule():
    import paper_2012_13618_amd as bp
    dhs = [bp.DeviceHypergraph.from_host(I.vlsi(seed=s, n=3000)) for s in range(3)]
    bp.profile_enable(True)
    try:
        bp.profile_reset()
        bp.partition_batch_device(dhs, [2, 4, 2], [0.05] * 3)
        one = sum(s["launches"] for s in bp.profile_read() if s["name"] == "batch")
        bp.profile_reset()
        best, ms = bp.autotune_batch_device(dhs, [2, 4, 2], [0.05] * 3, trials=1)
        runs = sum(s["launches"] for s in bp.profile_read() if s["name"] == "batch") / one
    finally:
        bp.profile_enable(False)
        bp.profile_reset()
    assert best.seg_select_max_nodes in (0, 4096, 16384) and ms > 0
    # the reference run, then 4 gain limits x 3 selection limits x 2 chunk lengths
    assert runs == 1 + 4 * 3 * 2
