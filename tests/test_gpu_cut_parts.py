"""The heaviest of very many parts: the loop over the part weights up to the
largest number of parts an int holds."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [511, 513, 1024 * 512 + 1, (1 << 31) - 512, (1 << 31) - 1])
def test_heaviest_part(k):
    import torch
    import paper_2012_13618_amd as bp
    n = 5000
    rng = np.random.default_rng(k % 1000)
    part = np.concatenate([rng.integers(0, k, n - 4), [k - 1, k - 1, 0, k // 2]]).astype(np.int32)
    w = np.concatenate([rng.integers(0, 3, n - 4), [50, 60, 7, 7]]).astype(np.int32)
    pins = rng.permutation(n).astype(np.int32)
    dh = bp.DeviceHypergraph(n, torch.arange(0, n + 1, 2, dtype=torch.int32).cuda(), torch.from_numpy(pins).cuda(),
                             torch.from_numpy(w).cuda(), None)
    try:
        cut, heavy = bp.compute_cut_device(dh, torch.from_numpy(part).cuda(), k)
    finally:
        bp.release_memory()
    ids, inv = np.unique(part, return_inverse=True)
    assert heavy == np.bincount(inv, weights=w).max()
    assert cut == int((part[pins[0::2]] != part[pins[1::2]]).sum())
