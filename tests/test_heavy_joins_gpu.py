"""Joins of long symbol lists cut into chunks over several workgroups, against
the oracle.

For a popped pair the arcs of both states are matched on every inner symbol
(Algorithm 2).  A source whose shorter list is longer than 2,048 symbols is
joined by up to 64 workgroups in whole steps of 512 symbols; its match and
record offsets continue across the chunks.  The list lengths below sit at the
edges of steps and chunks, the two lists of one length or one much longer, and
the middle state count exceeds the number of sources that are cut (256) so that
a level has sources of both kinds.
"""
import numpy as np
import pytest

import oracle
from fstcheck import assert_same, assert_same_multiset, canon_of, multiset_of
from paper_1805_06383_amd import workloads as W

pytestmark = pytest.mark.gpu


def pair(n1, n2, syms, width, seed):
    """State 0 goes to `width` states on symbols above the lists', each of
    which has a list of n1 (n2) symbols; M2's states loop to themselves."""
    rng = np.random.default_rng(seed)

    def one(n, inner_is_output):
        src, dst, inner, outer = [np.zeros(width, int)], [1 + np.arange(width)], \
            [syms + np.arange(width)], [rng.integers(0, 5, width)]
        for q in range(1, width + 1):
            src.append(np.full(n, q))
            dst.append(rng.integers(0, width + 1, n) if width < 8 else np.zeros(n, int))
            inner.append(np.sort(rng.choice(syms, n, replace=False)))
            outer.append(rng.integers(0, 5, n))
        src, dst, inner, outer = map(np.concatenate, (src, dst, inner, outer))
        g = syms + width
        il, ol, ni, no = (outer, inner, 5, g) if inner_is_output else (inner, outer, g, 5)
        return W.FST(width + 1, 0, ni, no, src, dst, il, ol, W.random_weights(rng, len(src)),
                     np.ones(width + 1, np.uint8))
    return one(n1, True), one(n2, False)


@pytest.mark.parametrize("reduce", [True, False])
@pytest.mark.parametrize("n1,n2,syms,width", [
    (2048, 2048, 4000, 2), (2049, 2049, 2049, 2), (2560, 2561, 3000, 3), (32768, 32768, 40000, 1),
    (32769, 33280, 33280, 1), (60000, 50001, 65000, 1), (2050, 2100, 2100, 300)])
def test_heavy_lists(n1, n2, syms, width, reduce):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1805_06383_amd import fstc
    m1, m2 = pair(n1, n2, syms, width, n1 + n2)
    cap = 2 if width > 3 else 4
    h = fstc.compose(m1, m2, max_levels=cap, reduce=reduce, deterministic_ids=True).to_host()
    ref = oracle.compose(m1, m2, max_levels=cap, reduce=reduce)
    if reduce:
        assert_same(canon_of(h), canon_of(ref), rtol=1e-5, what=f"{n1} {n2} {width}")
    else:
        assert_same_multiset(multiset_of(h), multiset_of(ref), what=f"{n1} {n2} {width}")
    assert h.num_premerge == ref.num_premerge


@pytest.mark.parametrize("n1,n2,syms,width", [
    (65, 65, 80, 1), (512, 513, 600, 3), (513, 2048, 2100, 512), (100, 511, 520, 513),
    (70, 90, 100, 1024), (66, 300, 310, 1025), (65, 66, 70, 8200)])
def test_wide_lists(n1, n2, syms, width):
    """Lists of 65 to 2,048 symbols: a workgroup per source up to the number of
    workgroups (512 and an eighth of the level to count, 1,024 to emit), a
    wavefront per source above."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1805_06383_amd import fstc
    m1, m2 = pair(n1, n2, syms, width, n1 + n2)
    for kw in (dict(deterministic_ids=True), dict(product=False)):
        h = fstc.compose(m1, m2, max_levels=2, small_levels=False, **kw).to_host()
        ref = oracle.compose(m1, m2, max_levels=2)
        assert_same(canon_of(h), canon_of(ref), rtol=1e-5, what=f"{n1} {n2} {width} {kw}")
        assert h.num_premerge == ref.num_premerge
