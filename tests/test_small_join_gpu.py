"""The one-workgroup levels' join at its lines, against the per-level kernels and
the oracle: more short-list symbols than threads (1,024), 1,024 and 1,025
joined pairs, 64 and 65 per source, lists of 32 and 33 symbols, empty lists
between others, long second lists, equal keys.

Algorithm 2 matches, composes, sorts and sums the arcs of every popped pair."""
import numpy as np
import pytest

import oracle
from fstcheck import assert_same, canon_of
from test_chunk_merge_gpu import layered

CASES = {
    "two-rounds": (22, [(3, 1), (3, 1), (2, 1)], [(4, 1), (3, 1)]),      # 484 x 2 to 3 symbols
    "records-1024": (4, [(1, 8)], [(1, 8)]),                             # 16 sources x 64
    "records-1025": (5, [(1, 8), (1, 8), (1, 8), (1, 8), (1, 1)], [(1, 8)] * 4 + [(1, 1)]),
    "per-source": (3, [(1, 8), (1, 5), (1, 9)], [(1, 8), (1, 13), (1, 7)]),
    "lists": (4, [(32, 1), (31, 1), (1, 1)], [(32, 1), (5, 1), (390, 1)]),
    "lists-33": (3, [(33, 1), (2, 1)], [(34, 1), (3, 1)]),
    "empty": (6, [(0, 1), (2, 1), (0, 1), (3, 2)], [(3, 1), (0, 1), (0, 1), (2, 2)]),
}


@pytest.mark.gpu
@pytest.mark.parametrize("distinct", [True, False])
@pytest.mark.parametrize("name", list(CASES))
def test_small_join(name, distinct):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1805_06383_amd import fstc
    width, s1, s2 = CASES[name]
    m1, m2 = layered(len(name), width, s1, s2, distinct=distinct)
    ref = oracle.compose(m1, m2)
    for kw in ({}, dict(deterministic_ids=True), dict(hash_visited=True)):
        h = fstc.compose(m1, m2, **kw).to_host()
        assert_same(canon_of(h), canon_of(ref), rtol=1e-5, what=f"{name} {kw}")
        assert h.num_premerge == ref.num_premerge
    y = fstc.compose(m1, m2, small_levels=False, deterministic_ids=True).to_host()
    g = fstc.compose(m1, m2, deterministic_ids=True).to_host()
    for f in ("q1", "q2", "final", "src", "dst", "a", "c"):
        assert np.array_equal(getattr(g, f), getattr(y, f)), f
    np.testing.assert_allclose(g.w, y.w, rtol=2.5e-7)
