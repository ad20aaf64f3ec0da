"""Composition without reduction of sparse machines over more than a million
pairs: levels of many sources number their new pairs in (q1, q2) order, which
keeps the next level's reads of rows and visited entries in order; others in the
order of claims.  Against the oracle, in both forms of the visited set.
"""
import numpy as np
import pytest

import oracle
from fstcheck import assert_same_multiset, multiset_of
from paper_1805_06383_amd import workloads as W


def sparse(n, degree, inner, seed):
    rng = np.random.default_rng(seed)

    def one(inner_is_output):
        a = n * degree
        src, dst = rng.integers(0, n, a), rng.integers(0, n, a)
        b, o = rng.integers(0, inner, a), rng.integers(0, 40, a)
        src[:30] = 0
        il, ol, ni, no = (o, b, 40, inner) if inner_is_output else (b, o, inner, 40)
        return W.FST(n, 0, ni, no, src, dst, il, ol, W.random_weights(rng, a),
                     (rng.random(n) < 0.2).astype(np.uint8))

    return one(True), one(False)


@pytest.mark.gpu
@pytest.mark.parametrize("kw", [{}, dict(hash_visited=True), dict(deterministic_ids=True)],
                         ids=["default", "hash", "ordered"])
@pytest.mark.parametrize("n", [1000, 1100])
def test_unreduced_sparse(n, kw):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1805_06383_amd import fstc
    m1, m2 = sparse(n, 8, 10, n)
    ref = oracle.compose(m1, m2, max_levels=5, reduce=False)
    h = fstc.compose(m1, m2, reduce=False, max_levels=5, **kw).to_host()
    assert_same_multiset(multiset_of(h), multiset_of(ref), what=f"{n} {kw}")
    assert h.num_premerge == ref.num_premerge == h.num_arcs
    sizes = np.bincount(ref.depth)
    first = np.cumsum(np.r_[0, sizes])
    key = h.q1.astype(np.uint64) * n + h.q2
    wide = 0
    for d in range(1, len(sizes)):  # the pairs found by the sources of depth d - 1
        ids = key[first[d]:first[d + 1]]
        if not kw and n * n > 1 << 20 and n * n <= 128 * sizes[d - 1]:
            wide += 1
            assert np.all(ids[1:] > ids[:-1])
        if kw.get("deterministic_ids"):
            assert np.all(ids[1:] > ids[:-1])
    if not kw and n * n > 1 << 20:
        assert wide >= 1
