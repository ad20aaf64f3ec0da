"""Levels that mix sources merged on the chip with a source of many joined
pairs, while the visited set is a hash table that has to grow for the latter.

A merged arc carries its target's slot in the visited set until the level's new
pairs have ids (Section 3.4, "Updating frontier and visited set"), so no slot
may be taken before the table has the size the level needs: a growth moves
every key, and the move into the dense array has other slots altogether.
"""
import numpy as np
import pytest

import oracle
from fstcheck import assert_same, canon_of
from paper_1805_06383_amd import workloads as W

# the visited set's start and the chunk merge's slots on a level of at most
# 4,096 sources (compose.hip): slots the claims may need before the general
# sources are counted
CHUNK_SLOTS = 256


def mixed_pair(seed, nq, width, hub, hub_arcs=2):
    """The start pair leads to (i, i) for i in 1..width, each with three sparse
    arcs a side, and to the pair (width + 1, width + 1) of `hub` arcs a side on
    one symbol of their own, to distinct targets; the other states have
    `hub_arcs` arcs each."""
    rng = np.random.default_rng(seed)

    def one(inner_is_output):
        kids = 1 + np.arange(width + 1)
        src, dst, inner = [np.zeros(width + 1, int)], [kids], [10 + kids]
        for i in range(1, width + 1):
            src.append(np.full(3, i))
            dst.append(rng.integers(width + 2, nq, 3))
            inner.append(rng.permutation(8)[:3])
        src.append(np.full(hub, width + 1))
        dst.append(nq - 1 - np.arange(hub))
        inner.append(np.full(hub, 8))
        rest = np.repeat(np.arange(width + 2, nq), hub_arcs)
        src.append(rest)
        dst.append(rng.integers(0, nq, len(rest)))
        inner.append(rng.integers(0, 8, len(rest)))
        src, dst, inner = map(np.concatenate, (src, dst, inner))
        out = rng.integers(0, 30, len(src))
        w = W.random_weights(rng, len(src))
        fin = (rng.random(nq) < 0.3).astype(np.uint8)
        ng = 12 + width + 1
        il, ol, ni, no = (out, inner, 30, ng) if inner_is_output else (inner, out, ng, 30)
        return W.FST(nq, 0, ni, no, src, dst, il, ol, w, fin)

    return one(True), one(False)


def pow2(x):
    return 1 << (int(x) - 1).bit_length()


# name: states a side, sparse pairs, arcs of the hub's symbol, depth cap
CASES = {"grow": (3500, 40, 150, 3), "grow-little": (3500, 33, 128, 3),
         "no-growth": (3500, 40, 60, 3), "sixty": (3000, 60, 200, 3)}
MOVE = (8250, 40, 2900, 2)


def sizes(m1, m2, nq, width, hub):
    """Slots of the first table, those the claims could need early, and those
    the level needs with the hub's pairs."""
    first = max(4096, pow2(2 * min(nq * nq, m1.num_arcs + m2.num_arcs + 1)))
    nsrc = width + 1
    return first, 2 * (1 + nsrc + nsrc * CHUNK_SLOTS), 2 * (1 + nsrc + hub * hub)


@pytest.mark.parametrize("name", list(CASES))
def test_inputs_reach_the_growth(name):
    """The inputs are what the tests below need: the second level has one hub
    among at least 32 sparse sources, the early claims fit the first table and
    (but for `no-growth`) the hub's do not."""
    nq, width, hub, cap = CASES[name]
    m1, m2 = mixed_pair(3, nq, width, hub)
    first, early, whole = sizes(m1, m2, nq, width, hub)
    assert width >= 32 and early <= first
    assert (whole > first) == (name != "no-growth")
    ref = oracle.compose(m1, m2, max_levels=2)
    second = np.flatnonzero(ref.depth == 1)
    assert len(second) == width + 1
    out = np.bincount(ref.src, minlength=ref.num_states)[second]
    assert sorted(out)[-1] == hub * hub and 0 < sum(sorted(out)[:-1]) <= 9 * width


def test_inputs_reach_the_move():
    nq, width, hub, cap = MOVE
    pairs = nq * nq
    assert (1 << 26) < pairs <= (1 << 30)
    m1, m2 = mixed_pair(4, nq, width, hub)
    first, early, whole = sizes(m1, m2, nq, width, hub)
    assert early <= first < whole and pow2(whole) * 12 >= pairs * 4


def composed(m1, m2, cap, **kw):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1805_06383_amd import fstc
    g = fstc.compose(m1, m2, max_levels=cap, **kw)
    # both merges ran
    assert g.stats["total_product_records"] > 0 and g.stats["total_matches"] > 0
    return g


@pytest.mark.gpu
@pytest.mark.parametrize("ordered", [False, True])
@pytest.mark.parametrize("small", [False, True])
@pytest.mark.parametrize("name", list(CASES))
def test_mixed_level_grows_the_table(name, small, ordered):
    nq, width, hub, cap = CASES[name]
    m1, m2 = mixed_pair(3, nq, width, hub)
    ref = oracle.compose(m1, m2, max_levels=cap)
    g = composed(m1, m2, cap, hash_visited=True, deterministic_ids=ordered, small_levels=small)
    assert g.stats["visited_form"] == 0
    h = g.to_host()
    assert_same(canon_of(h), canon_of(ref), rtol=1e-5, what=f"{name} {ordered}")
    assert h.num_premerge == ref.num_premerge
    if ordered:  # the same arrays as over the dense visited set
        d = composed(m1, m2, cap, deterministic_ids=True, small_levels=small).to_host()
        for f in ("q1", "q2", "final", "src", "dst", "a", "c", "w"):
            assert np.array_equal(getattr(h, f), getattr(d, f)), f


@pytest.mark.gpu
@pytest.mark.timeout(300)
def test_mixed_level_moves_the_table():
    """The same where the grown table would be no smaller than the dense array."""
    nq, width, hub, cap = MOVE
    m1, m2 = mixed_pair(4, nq, width, hub)
    ref = canon_of(oracle.compose(m1, m2, max_levels=cap))
    for ordered in (False, True):
        g = composed(m1, m2, cap, deterministic_ids=ordered)
        assert g.stats["visited_form"] == 2
        assert_same(canon_of(g.to_host()), ref, rtol=1e-5, what=f"move {ordered}")
