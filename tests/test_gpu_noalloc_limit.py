"""Calls near the fixed workspace's limit that it holds: many nodes, hardly any
hyperedges, and windowed balance rounds on several tree levels."""
import pytest

pytestmark = pytest.mark.gpu


def graph(n, e):
    import torch
    import paper_2012_13618_amd as bp
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    deg = torch.randint(2, 5, (e,), device="cuda", generator=g)
    off = torch.zeros(e + 1, dtype=torch.int64, device="cuda")
    off[1:] = torch.cumsum(deg, 0)
    he = torch.repeat_interleave(torch.arange(e, device="cuda"), deg)
    start = torch.randint(0, n, (e,), device="cuda", generator=g)
    # (7919 is prime and no divisor of n: the pins of a hyperedge differ)
    pins = (start[he] + (torch.arange(len(he), device="cuda") - off[he]) * 7919) % n
    return bp.DeviceHypergraph(n, off.int(), pins.int(), None, None)


@pytest.mark.parametrize("n,e,k", [(1965744, 500, 2), (966858, 5000, 3), (609407, 5000, 8), (458954, 5000, 16),
                                   (389210, 500, 32), (357373, 5000, 32), (289652, 5000, 64)])
def test_fits(n, e, k):
    import torch
    import paper_2012_13618_amd as bp
    dh = graph(n, e)
    part = torch.empty(n, dtype=torch.int32, device="cuda")
    _, cut, _, rep = bp.partition_device_noalloc(dh, k, 0.05, part_out=part)
    assert rep.device_bytes <= 256 << 20
    ref, rcut, _, _ = bp.partition_device(dh, k, 0.05)
    assert cut == rcut and torch.equal(part, ref)
