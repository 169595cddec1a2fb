"""Cut and part weights at the sizes where the cut kernel's ways change: a tile
of 512 hyperedges, 32 pins (thread or wavefront), 4096 (workgroup, past their
queue), 64 parts (bit mask or scan) and 2^19 nodes (parts as bytes); and an
input that fails its check."""
import numpy as np
import pytest

import oracle
from paper_2012_13618_amd import inputs as I

pytestmark = pytest.mark.gpu


def graph(n, degs, seed):
    rng = np.random.default_rng(seed)
    degs = np.asarray(degs)
    off = np.concatenate([[0], np.cumsum(degs)])
    start = rng.integers(0, n, len(degs))
    pins = (np.repeat(start - off[:-1], degs) + np.arange(off[-1])) % n
    return I.Hypergraph(n, off.astype(np.int32), pins.astype(np.int32), rng.integers(1, 4, n).astype(np.int32),
                        rng.integers(0, 5, len(degs)).astype(np.int32))


def sizes(kind):
    rng = np.random.default_rng(3)
    if kind == "edges":
        return np.tile([0, 1, 2, 8, 9, 31, 32, 33, 64, 65, 512, 513], 171)
    if kind == "huge":  # past the workgroups' queue, and a full wavefront queue
        return np.concatenate([np.full(100, 4096), np.full(600, 33), [4095, 4097, 9000], np.full(50, 2)])
    if kind == "many":  # several tiles a workgroup
        return rng.integers(0, 6, 1300000)
    return np.full(int(kind), 2)


@pytest.mark.parametrize("n,kind,k", [
    (1, "1", 2), (700, "511", 1), (700, "513", 3), (10000, "edges", 64), (10000, "edges", 65), (10000, "huge", 16),
    (3000, "edges", 5000), ((1 << 19) - 1, "many", 2), (1 << 19, "many", 2), (1 << 19, "edges", 64),
    (1 << 19, "huge", 65), ((1 << 19) + 3, "many", 33),
])
@pytest.mark.parametrize("weights", [True, False])
def test_cut(n, kind, k, weights):
    import torch
    import paper_2012_13618_amd as bp
    h = graph(n, np.minimum(sizes(kind), n), n % 1000)
    part = np.random.default_rng(k).integers(0, k, n).astype(np.int32)
    if not weights:
        h.node_w, h.hedge_w = None, None
    dh = bp.DeviceHypergraph(n, torch.from_numpy(h.offsets).cuda(), torch.from_numpy(h.pins).cuda(),
                             None if h.node_w is None else torch.from_numpy(h.node_w).cuda(),
                             None if h.hedge_w is None else torch.from_numpy(h.hedge_w).cuda())
    cut, heavy = bp.compute_cut_device(dh, torch.from_numpy(part).cuda(), k)
    w = np.ones(n, np.int64) if h.node_w is None else h.node_w
    assert heavy == np.bincount(part, weights=w, minlength=k).max()
    # distinct parts per hyperedge
    he = np.repeat(np.arange(len(h.offsets) - 1), np.diff(h.offsets)).astype(np.int64)
    lam = np.bincount(np.unique(he * k + part[h.pins]) // k, minlength=len(h.offsets) - 1)
    hw = np.ones(len(lam), np.int64) if h.hedge_w is None else h.hedge_w
    assert cut == int((hw * np.maximum(lam - 1, 0)).sum())


def test_refused():
    """A pin out of range is an error, and nothing is read through it."""
    import torch
    import paper_2012_13618_amd as bp
    for bad in (-1, 100):
        pins = np.tile(np.array([0, 1, 99], np.int32), 400)
        pins[700] = bad
        dh = bp.DeviceHypergraph(100, torch.arange(0, 1201, 3, dtype=torch.int32).cuda(),
                                 torch.from_numpy(pins).cuda(), None, None)
        with pytest.raises(bp.BipartError):
            bp.compute_cut_device(dh, torch.zeros(100, dtype=torch.int32).cuda(), 2)
