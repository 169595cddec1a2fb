"""The per-pin hyperedge ids and the pin copies taken in tiles of 4096 pins:
matching (node-major incidence) and coarsening (copied lists, then the coarse
level's incidence) exact against the oracle where tiles begin and end."""
import numpy as np
import pytest

import oracle
from paper_2012_13618_amd import inputs as I

pytestmark = pytest.mark.gpu
T = 4096


@pytest.fixture(scope="module")
def bp():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2012_13618_amd as mod
    mod.lib()
    return mod


def graph(n, deg, seed):
    rng = np.random.default_rng(seed)
    off = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    start = rng.integers(0, n, len(deg))
    pins = (np.repeat(start - off[:-1], deg) + np.arange(off[-1])) % n
    return I.Hypergraph(n, off, pins.astype(np.int32), np.ones(n, np.int32), np.ones(len(deg), np.int32))


DEGREES = {
    "one tile less a pin": [2] * (T // 2 - 1) + [1],
    "one tile": [2] * (T // 2),
    "one pin more": [2] * (T // 2) + [1],
    "a hyperedge over a tile's end": [2] * (T // 2 - 1) + [3, 2],
    "tiles inside one hyperedge": [5, 3 * T + 7, 2],
    "starts at tile starts": [T, T, 2 * T, 3],
    "empty ones at the ends": [0, 0, T - 1, 0, 1, 0, 0, T, 0, 4, 0],
    "mixed": list(np.random.default_rng(1).integers(0, 60, 3000)),
}


@pytest.mark.parametrize("name", DEGREES)
def test_match(bp, name):
    h = graph(4 * T, np.array(DEGREES[name]), 3)
    got = bp.step_match(bp.DeviceHypergraph.from_host(h)).cpu().numpy()
    assert np.array_equal(got, oracle.match(h.num_nodes, h.offsets, h.pins, hw=h.hedge_w))


def test_match_single_node(bp):
    h = I.Hypergraph(1, np.arange(4, dtype=np.int32), np.zeros(3, np.int32), np.ones(1, np.int32),
                     np.ones(3, np.int32))
    got = bp.step_match(bp.DeviceHypergraph.from_host(h)).cpu().numpy()
    assert np.array_equal(got, oracle.match(1, h.offsets, h.pins, hw=h.hedge_w))


@pytest.mark.parametrize("name", [k for k in DEGREES if "empty" not in k and k != "mixed"])
@pytest.mark.parametrize("n", [4 * T, 9 * T])
def test_coarsen_then_partition(bp, name, n):
    deg = np.maximum(np.array(DEGREES[name]), 2)
    h = graph(n, np.concatenate([deg, np.random.default_rng(5).integers(2, 9, 6000)]), n)
    got = [t.cpu().numpy() for t in bp.step_coarsen(bp.DeviceHypergraph.from_host(h))]
    ref = oracle.coarsen(n, h.offsets, h.pins, h.node_w, h.hedge_w)
    for what, a, b in zip(["parent", "offsets", "pins", "node_w", "hedge_w"], got, ref):
        assert np.array_equal(a, b), what
    part, cut, _, _ = bp.partition_device(bp.DeviceHypergraph.from_host(h), 3, 0.05)
    want, want_cut = oracle.partition(n, h.offsets, h.pins, 3, 0.05)
    assert np.array_equal(part.cpu().numpy(), want) and cut == want_cut
