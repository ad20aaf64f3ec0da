"""Ordered state ids (deterministic_ids) in every form they are given in:
ranked in one launch, by a pass over the dense visited array, by a sort of the
hash table's new pairs, and by the direct product levels, against the oracle's
states sorted by depth and pair.

The start pair joins h1 x h2 arcs to as many distinct target pairs, so that the
number of new pairs sits at the edges of the ranked form (tiles of 2,048, at
most 16,384); every target has one more arc, so that a second level follows.
"""
import numpy as np
import pytest

import oracle
from fstcheck import assert_same, assert_same_multiset, canon_of, multiset_of
from paper_1805_06383_amd import workloads as W

pytestmark = pytest.mark.gpu


def hubs(h1, h2, nq1, nq2, seed=0):
    rng = np.random.default_rng(seed)

    def one(inner_is_output, h, nq):
        t = 1 + rng.permutation(nq - 1)[:h]
        src = np.r_[np.zeros(h, int), 1 + np.arange(nq - 1)]
        dst = np.r_[t, rng.integers(0, nq, nq - 1)]
        inner = np.r_[np.zeros(h, int), rng.integers(0, 3, nq - 1)]
        outer = rng.integers(0, 7, len(src))
        il, ol, ni, no = (outer, inner, 7, 3) if inner_is_output else (inner, outer, 3, 7)
        return W.FST(nq, 0, ni, no, src, dst, il, ol, W.random_weights(rng, len(src)),
                     (rng.random(nq) < 0.5).astype(np.uint8))
    return one(True, h1, nq1), one(False, h2, nq2)


def check_order(h, nq2):
    depth = np.full(h.num_states, -1)
    depth[0] = 0
    for _ in range(h.num_states):
        new = (depth[h.src] >= 0) & (depth[h.dst] < 0)
        if not new.any():
            break
        d = depth[h.src[new]].min()
        depth[h.dst[new & (depth[h.src] == d)]] = d + 1
    assert np.all(depth >= 0)
    key = depth.astype(np.int64) << 40 | h.q1.astype(np.int64) * nq2 + h.q2
    assert np.all(key[1:] > key[:-1]), "ids are not in (depth, q1, q2) order"


def compose(m1, m2, **kw):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1805_06383_amd import fstc
    return fstc.compose(m1, m2, deterministic_ids=True, **kw)


SIZES = [(1, 1), (3, 21), (8, 8), (5, 13), (32, 64), (683, 3), (127, 129), (128, 128), (128, 129),
         (300, 300)]


@pytest.mark.parametrize("form", ["scan", "dense", "hash", "capped", "unreduced", "unreduced-hash"])
@pytest.mark.parametrize("h1,h2", SIZES)
def test_hub_levels(h1, h2, form):
    n = 700 if form != "dense" else 2300  # pair spaces below and above 2^22
    kw = {"scan": {}, "dense": {}, "hash": dict(hash_visited=True), "capped": dict(max_arcs=1 << 30),
          "unreduced": dict(reduce=False),
          "unreduced-hash": dict(reduce=False, hash_visited=True)}[form]
    m1, m2 = hubs(h1, h2, n, n + 1, seed=h1 * 1000 + h2)
    h = compose(m1, m2, small_levels=False, **kw).to_host()
    ref = oracle.compose(m1, m2, reduce=kw.get("reduce", True))
    check_order(h, m2.num_states)
    if kw.get("reduce", True):
        assert_same(canon_of(h), canon_of(ref), rtol=1e-5, what=f"{h1}x{h2} {form}")
    else:
        assert_same_multiset(multiset_of(h), multiset_of(ref), what=f"{h1}x{h2} {form}")


@pytest.mark.parametrize("nq,h1,h2", [(7400, 160, 130), (8000, 160, 130)])
def test_pass_or_sort(nq, h1, h2):
    """More new pairs than are ranked, over a dense visited array on both sides
    of the size from which their sort is cheaper than a pass over it."""
    m1, m2 = hubs(h1, h2, nq, nq + 1)
    h = compose(m1, m2).to_host()
    check_order(h, m2.num_states)
    assert_same(canon_of(h), canon_of(oracle.compose(m1, m2)), rtol=1e-5, what=f"{nq}")


@pytest.mark.parametrize("slots", [1, 3, 4])
@pytest.mark.parametrize("nq,m", [(3, 8), (9, 8), (40, 64), (70, 33)])
def test_direct_product_levels(nq, m, slots):
    """Levels of at most 64 pairs (one workgroup, with the small levels on)
    and above."""
    m1, m2 = W.config4(nq + slots, nq=nq, m=m, slots=slots)
    ref = oracle.compose(m1, m2)
    a = compose(m1, m2)
    b = compose(m1, m2, small_levels=False)
    assert b.stats["direct_product_levels"] > 0 and b.stats["group_product_levels"] == 0
    assert m < 33 or a.stats["group_product_levels"] > 0
    for r in (a, b):
        h = r.to_host()
        check_order(h, m2.num_states)
        assert_same(canon_of(h), canon_of(ref), rtol=1e-5, what=f"{nq} {m} {slots}")
    x, y = a.to_host(), b.to_host()
    for f in ("q1", "q2", "final", "src", "dst", "a", "c"):
        assert np.array_equal(getattr(x, f), getattr(y, f)), f


@pytest.mark.parametrize("slots", [1, 2, 3, 4])
@pytest.mark.parametrize("nq,m", [(7, 8), (20, 33), (40, 64)])
def test_unreduced_product_order(nq, m, slots):
    """Without reduction, strided sources write their joined pairs from the
    two weight matrices in the order of the written records: the same arrays,
    bit for bit, as with every source on records."""
    m1, m2 = W.config4(nq * slots, nq=nq, m=m, slots=slots)
    a = compose(m1, m2, reduce=False)
    b = compose(m1, m2, reduce=False, product=False)
    assert a.stats["total_product_records"] > 0  # not all: a state may hold a slot twice
    assert b.stats["total_product_records"] == 0
    x, y = a.to_host(), b.to_host()
    for f in ("q1", "q2", "final", "src", "dst", "a", "c", "w"):
        assert np.array_equal(getattr(x, f), getattr(y, f)), f
