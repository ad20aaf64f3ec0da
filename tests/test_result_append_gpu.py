"""The result append on levels that mix multi-block, tile-merged and
product-merge sources, against the oracle.

Algorithm 2 appends the merged arcs of a level's pairs to the composition
(Section 3.4).  Merge tiles and multi-block sources are copied by several
waves each, and on levels with product-merge sources in between every run goes
to its own source's place.  The pairs below hold, in one search: hub states
with one inner symbol (a pair of them is one multi-block source of hub1 x hub2
arcs, its size around the copied chunks of 256), dense states (product-merge
sources) and irregular ones (tiles).
"""
import numpy as np
import pytest

import oracle
from fstcheck import assert_same, canon_of
from paper_1805_06383_amd import workloads as W

NQ, SYMS = 48, 32


def mixed_pair(seed, hub1, hub2):
    rng = np.random.default_rng(seed)

    def one(inner_is_output, hub):
        src, dst, inner, outer = [], [], [], []

        def add(q, d, b, o):
            src.append(np.full(len(d), q)), dst.append(d), inner.append(b), outer.append(o)

        for q in [0] + list(range(40, NQ)):            # hubs: every arc on symbol 0
            add(q, 1 + np.arange(hub) % (NQ - 1), np.zeros(hub, int), np.arange(hub))
        for q in range(1, 24):                         # dense: three slots x all symbols
            add(q, np.tile(rng.integers(0, NQ, 3), SYMS), np.repeat(np.arange(SYMS), 3),
                np.tile(rng.choice(hub, 3, replace=False), SYMS))
        for q in range(24, 40):                        # irregular
            n = int(rng.integers(1, 40))
            add(q, rng.integers(0, NQ, n), rng.integers(0, SYMS, n), rng.integers(0, hub, n))
        src, dst, inner, outer = map(np.concatenate, (src, dst, inner, outer))
        p = rng.permutation(len(src))
        src, dst, inner, outer = src[p], dst[p], inner[p], outer[p]
        il, ol, ni, no = (outer, inner, hub, SYMS) if inner_is_output else (inner, outer, SYMS, hub)
        return W.FST(NQ, 0, ni, no, src, dst, il, ol, W.random_weights(rng, len(src)),
                     (rng.random(NQ) < 0.3).astype(np.uint8))
    return one(True, hub1), one(False, hub2)


@pytest.mark.gpu
@pytest.mark.parametrize("mode", ["default", "ordered", "records", "capped", "hash"])
@pytest.mark.parametrize("hub1,hub2", [(46, 45), (64, 64), (61, 67), (130, 190)])
def test_mixed_levels(hub1, hub2, mode):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1805_06383_amd import fstc
    kw = {"default": {}, "ordered": dict(deterministic_ids=True), "records": dict(product=False),
          "capped": dict(max_levels=2), "hash": dict(hash_visited=True, deterministic_ids=True)}[mode]
    m1, m2 = mixed_pair(hub1, hub1, hub2)
    g = fstc.compose(m1, m2, **kw)
    ref = oracle.compose(m1, m2, max_levels=kw.get("max_levels", 0))
    assert g.stats["big_sources"] > 0 and (mode == "records" or g.stats["total_product_sources"] > 0)
    h = g.to_host()
    assert_same(canon_of(h), canon_of(ref), rtol=1e-5, what=f"{hub1} x {hub2} {mode}")
    assert np.all(h.src[1:] >= h.src[:-1])
    if kw.get("deterministic_ids"):
        depth = np.zeros(h.num_states, int)            # ids by depth, then by pair
        for s, d in zip(h.src, h.dst):
            if d > 0 and depth[d] == 0:
                depth[d] = depth[s] + 1
        key = depth * NQ * NQ + h.q1.astype(int) * NQ + h.q2
        assert np.all(key[1:] > key[:-1])
