"""How a cut's large hyperedges are shared out: the runs of hyperedges that make
a workgroup's tile, the list that those of more than 32 pins go to above 64
parts, and that neither few large hyperedges nor many parts leave the card to a
few workgroups."""
import time

import numpy as np
import pytest

from paper_2012_13618_amd import inputs as I

pytestmark = pytest.mark.gpu


def graph(n, degs):
    degs = np.asarray(degs)
    off = np.concatenate([[0], np.cumsum(degs)])
    start = np.random.default_rng(n).integers(0, n, len(degs))
    # (7919 is prime and no divisor of n: the pins of a hyperedge differ)
    pins = (np.repeat(start, degs) + (np.arange(off[-1]) - np.repeat(off[:-1], degs)) * 7919) % n
    return I.Hypergraph(n, off.astype(np.int32), pins.astype(np.int32), np.ones(n, np.int32),
                        np.random.default_rng(n + 1).integers(0, 5, len(degs)).astype(np.int32))


def parts(n, k):
    return np.random.default_rng(k).integers(0, k, n).astype(np.int32)


def check(h, k):
    import torch
    import paper_2012_13618_amd as bp
    part = parts(h.num_nodes, k)
    cut, heavy = bp.compute_cut_device(bp.DeviceHypergraph.from_host(h), torch.from_numpy(part).cuda(), k)
    he = np.repeat(np.arange(len(h.hedge_w)), np.diff(h.offsets)).astype(np.int64)
    lam = np.bincount(np.unique(he * k + part[h.pins]) // k, minlength=len(h.hedge_w))
    assert cut == int((h.hedge_w.astype(np.int64) * np.maximum(lam - 1, 0)).sum())
    assert heavy == np.bincount(part, minlength=k).max()


# one run or several a workgroup, whole tiles, and ragged ends of each
@pytest.mark.parametrize("k", [3, 65])
@pytest.mark.parametrize("e", [1, 7, 9, 2047, 2049, 4100, 65535, 131071, 131072 + 65, 524288 + 3])
def test_runs(e, k):
    check(graph(30011, np.random.default_rng(e).integers(0, 40 if e < 10000 else 5, e)), k)


# a tile of large ones only, both ends of the list, and its two kinds' edge
@pytest.mark.parametrize("k", [16, 64, 65, 300, 20000])
@pytest.mark.parametrize("degs", [
    [256, 257] * 600, [33] * 1500, [257] * 1500, [4095, 4096, 4097, 2, 256, 33, 32] * 30, [0] * 700 + [300] + [0] * 700,
], ids=["mixed", "front", "back", "sizes", "lone"])
def test_list(degs, k):
    check(graph(20011, degs), k)


@pytest.mark.parametrize("name,degs", [("few", [2000] * 512), ("together", [4000] * 300 + [2] * 300000)])
@pytest.mark.parametrize("k", [16, 128])
def test_large_ones_are_shared_out(name, degs, k):
    """A million pins in few hyperedges, alone or side by side, against as many in
    hyperedges of four: by one workgroup 16 and 700 times as long."""
    import torch
    import paper_2012_13618_amd as bp
    n = 100003
    part = torch.from_numpy(parts(n, k)).cuda()

    def best(degs):
        dh = bp.DeviceHypergraph.from_host(graph(n, degs))
        t = []
        for _ in range(12):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            bp.compute_cut_device(dh, part, k)
            t.append(time.perf_counter() - t0)
        return min(t)

    small, large = best([4] * (int(np.sum(degs)) // 4)), best(degs)
    print(f"{name} k={k}: {1e6 * large:.0f} us, hyperedges of four {1e6 * small:.0f} us", flush=True)
    assert large < (6 if k <= 64 else 100) * small
