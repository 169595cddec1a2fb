"""The report's count of refined pins: every swap round's gain pass, on the small
levels that share a launch as on the others."""
import pytest

from paper_2012_13618_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h", [I.tiny(), I.vlsi(seed=4, n=6000)], ids=["tiny", "netlist"])
def test_pins_refined(h):
    import paper_2012_13618_amd as bp
    dh = bp.DeviceHypergraph.from_host(h)
    got = [bp.partition_device(dh, 2, 0.05, bp.params(refine_iters=it))[3].pins_refined for it in range(4)]
    # (coarsening, and so the levels' pins, do not hang on the rounds)
    assert got[0] == 0 and got[1] > 0 and got == [it * got[1] for it in range(4)], got
