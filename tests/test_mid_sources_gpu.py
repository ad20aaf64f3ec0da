"""Sources of more records than a merge tile takes: up to 8,192 records sorted
by a workgroup each, above that by the multi-block sort, against the oracle and
with ordered ids against a second run's arrays.

Algorithm 2 sorts and sums the arcs of every popped pair (Section 3.4).  The
counts sit at both lines (2,048 and 8,192 records), with nearly all keys
distinct and with few keys, and with part ranks of 32 bits and more.
"""
import numpy as np
import pytest

import oracle
from fstcheck import assert_same, canon_of
from paper_1805_06383_amd import workloads as W
from test_chunk_merge_gpu import layered

# arcs on the one shared symbol: products 2,047 to 2,049, 8,191 to 8,193 and more
SPEC1 = [(1, 64), (1, 3), (1, 1)]
SPEC2 = [(1, 128), (1, 2731), (1, 8191), (1, 683), (1, 32), (1, 2047)]


def wide_parts(m, inner_is_output, seed):
    """The transducer with a state that nothing reaches and 2^17 parts."""
    n = 1 << 17
    rng = np.random.default_rng(seed)
    z = np.full(n, m.num_states)
    il, ol = (np.arange(n), np.zeros(n, int)) if inner_is_output else (np.zeros(n, int), np.arange(n))
    cat = lambda a, b: np.concatenate([np.asarray(a), b])
    return W.FST(m.num_states + 1, m.start, max(m.num_isyms, n) if inner_is_output else m.num_isyms,
                 m.num_osyms if inner_is_output else max(m.num_osyms, n), cat(m.src, z),
                 cat(m.dst, z), cat(m.ilabel, il), cat(m.olabel, ol),
                 cat(m.weight, W.random_weights(rng, n)), np.r_[m.final, np.uint8(0)].astype(np.uint8))


@pytest.mark.gpu
@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("distinct", [True, False])
def test_mid_sources(distinct, wide):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1805_06383_amd import fstc
    m1, m2 = layered(3, 6, SPEC1, SPEC2, syms=2, outer=5000 if distinct else 50, distinct=distinct)
    if wide:
        m1, m2 = wide_parts(m1, True, 1), wide_parts(m2, False, 2)
    ref = oracle.compose(m1, m2, max_levels=2)
    for kw in ({}, dict(deterministic_ids=True), dict(hash_visited=True), dict(fused=True),
               dict(max_arcs=1 << 40)):
        g = fstc.compose(m1, m2, max_levels=2, **kw)
        assert g.stats["big_sources"] > 0 and g.stats["total_big_records"] > 0
        h = g.to_host()
        assert_same(canon_of(h), canon_of(ref), rtol=1e-5, what=f"{distinct} {wide} {kw}")
        assert h.num_premerge == ref.num_premerge
        if kw.get("deterministic_ids"):  # sums in a fixed order: the same bits again
            y = fstc.compose(m1, m2, max_levels=2, **kw).to_host()
            for f in ("q1", "q2", "final", "src", "dst", "a", "c", "w"):
                assert np.array_equal(getattr(h, f), getattr(y, f)), f
