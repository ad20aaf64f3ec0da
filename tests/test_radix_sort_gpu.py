"""The stable radix sort (section 3.4 sorts packed keys with a library call) at
the lines between its forms: one workgroup up to 8,192 pairs, tiles of 2,048
pairs up to 2^20 and of 4,096 above; pass counts of 1 to 8, even and odd; keys of
few values, where every tile adds to the same digits, and a caller's repeated
sorts.  Whole numbers: the order is numpy's stable order exactly."""
import numpy as np
import pytest


def check(n, lo, hi, values, seed):
    import torch
    from paper_1805_06383_amd import fstc as F
    rng = np.random.default_rng(seed)
    keys = rng.integers(0, 1 << 62, size=n, dtype=np.int64)
    if values:
        keys = rng.integers(0, 1 << 62, size=values, dtype=np.int64)[rng.integers(0, values, n)]
    if hi < 64:
        keys &= (1 << hi) - 1
    k, v = torch.from_numpy(keys.copy()).cuda(), torch.arange(n, dtype=torch.int32, device="cuda")
    F.fstc_sort_pairs(k, v, lo, hi)
    width = hi - lo
    field = keys.view(np.uint64) >> np.uint64(lo)
    if width < 64:
        field &= np.uint64((1 << width) - 1)
    order = np.argsort(field, kind="stable")
    assert np.array_equal(v.cpu().numpy(), order.astype(np.int32)), (n, lo, hi, values)
    assert np.array_equal(k.cpu().numpy(), keys[order]), (n, lo, hi, values)


@pytest.mark.gpu
@pytest.mark.parametrize("n", [2, 63, 64, 8191, 8192, 8193, 10_240, 10_241, (1 << 20) - 1, 1 << 20,
                               (1 << 20) + 1, 3_000_001])
@pytest.mark.parametrize("lo,hi", [(0, 1), (3, 11), (0, 17), (5, 30), (0, 33), (1, 64)])
def test_radix_sizes(n, lo, hi):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    for values in (0, 1, 3):
        check(n, lo, hi, values, n + hi)
