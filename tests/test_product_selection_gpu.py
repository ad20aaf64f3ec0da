"""Which sources the product merge takes on levels that the on-chip merge is
tried on: every source whose sums the matrix cores form from exact float64
products keeps that form, whatever the start state and the level's other
sources are (its results are then the sums rounded once).

The paper merges a source's arcs by sorting and summing them (Section 3.4); a
source whose two states have single-arc cells is merged as a small matrix
product instead, with no rounding of the products.
"""
import numpy as np
import pytest

from paper_1805_06383_amd import workloads as W


def machine(seed, inner_is_output, dense, sparse, slots, syms, kids, wide=0, base=0):
    """State 0 leads to states 1..kids, each by a symbol of its own.  States
    1..dense have `slots` (outer symbol, target) pairs and one arc to each for
    every one of the first `syms` symbols (the first `wide` if given).  The
    `sparse` states after them have two arcs.  The symbols of state 0 begin at
    `base` (by default, at `syms`)."""
    rng = np.random.default_rng(seed)
    n = 1 + dense + sparse
    base = base or syms
    d = np.arange(1, dense + 1)
    k = 1 + np.arange(kids) * (n - 1) // kids
    src, dst, inner, out = [np.zeros(kids, int)], [k], [base + np.arange(kids)], [np.zeros(kids, int)]
    m = wide or syms
    tgt = 1 + rng.integers(0, n - 1, (dense, slots))
    o = (rng.integers(0, 50, (dense, 1)) + np.arange(slots)) % 50  # distinct parts
    src.append(np.repeat(d, m * slots))
    inner.append(np.tile(np.repeat(np.arange(m), slots), dense))
    dst.append(np.tile(tgt[:, None, :], (1, m, 1)).ravel())
    out.append(np.tile(o[:, None, :], (1, m, 1)).ravel())
    s = np.repeat(np.arange(dense + 1, n), 2)
    src.append(s)
    dst.append(1 + rng.integers(0, n - 1, len(s)))
    inner.append(rng.integers(0, syms, len(s)))
    out.append(rng.integers(0, 50, len(s)))
    src, dst, inner, out = map(np.concatenate, (src, dst, inner, out))
    w = (rng.integers(1 << 23, 1 << 24, len(src)) / (1 << 24)).astype(np.float32)
    il, ol, ni, no = (out, inner, 50, base + kids) if inner_is_output else \
        (inner, out, base + kids, 50)
    fin = (rng.random(n) < 0.3).astype(np.uint8)
    return W.FST(n, 0, ni, no, src, dst, il, ol, w, fin)


def rows(m, inner, outer):
    """Float64 weights by (state, target, outer symbol) and inner symbol."""
    key = np.stack([m.src, m.dst, outer], 1).astype(np.int64)
    u, r = np.unique(key, axis=0, return_inverse=True)
    x = np.zeros((len(u), int(inner.max()) + 1))
    np.add.at(x, (r.ravel(), inner.astype(np.int64)), m.weight.astype(np.float64))
    return {tuple(k): i for i, k in enumerate(u.tolist())}, x


def exact(m1, m2, h, arcs):
    """The sums over the inner symbols of the result arcs `arcs`, in float64."""
    r1, x1 = rows(m1, m1.olabel, m1.ilabel)
    r2, x2 = rows(m2, m2.ilabel, m2.olabel)
    q1, q2 = h.q1.astype(np.int64), h.q2.astype(np.int64)
    i1 = [r1[k] for k in zip(q1[h.src[arcs]].tolist(), q1[h.dst[arcs]].tolist(), h.a[arcs].tolist())]
    i2 = [r2[k] for k in zip(q2[h.src[arcs]].tolist(), q2[h.dst[arcs]].tolist(), h.c[arcs].tolist())]
    n = min(x1.shape[1], x2.shape[1])
    return np.einsum("ij,ij->i", x1[i1, :n], x2[i2, :n])


# dense, sparse states, slots, symbols of the dense states
CASES = {"dense": (60, 0, 4, 8), "pairs-32": (60, 0, 2, 8), "half": (30, 30, 4, 12),
         "few": (12, 48, 3, 9), "pairs-256": (40, 20, 4, 16)}


def check(m1, m2, dense, cap=0, **kw):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1805_06383_amd import fstc
    g = fstc.compose(m1, m2, max_levels=cap, small_levels=False, **kw)
    h = g.to_host()
    both = (h.q1 >= 1) & (h.q1 <= dense) & (h.q2 >= 1) & (h.q2 <= dense)
    assert 0 < np.count_nonzero(both)
    if not cap:
        assert g.stats["total_product_mfma_sources"] == np.count_nonzero(both)
    arcs = np.flatnonzero(both[h.src])
    arcs = arcs[:: max(1, len(arcs) // 20000)]
    ref = exact(m1, m2, h, arcs)
    # one rounding to float32 of a float64 sum of at most 64 exact terms
    assert np.all(np.abs(h.w[arcs] - ref) <= 2.0**-24 * (1 + 1e-6) * ref)
    return g


@pytest.mark.gpu
@pytest.mark.parametrize("mode", [{}, dict(deterministic_ids=True), dict(hash_visited=True)],
                         ids=["default", "ordered", "hash"])
@pytest.mark.parametrize("name", list(CASES))
def test_exact_products_behind_a_wide_start(name, mode):
    dense, sparse, slots, syms = CASES[name]
    m1 = machine(1, True, dense, sparse, slots, syms, 40)
    m2 = machine(2, False, dense, sparse, slots, syms, 40)
    g = check(m1, m2, dense, **mode)
    if not sparse and not mode:  # levels of such sources alone are direct again
        assert g.stats["direct_product_levels"] >= 2


@pytest.mark.gpu
def test_full_cells_of_more_parts():
    """Five parts a side, 200 pairs on 25 entries: not for the matrix cores, and
    much dearer merged pair by pair."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle
    from fstcheck import assert_same, canon_of
    from paper_1805_06383_amd import fstc
    m1, m2 = machine(1, True, 40, 0, 5, 8, 40), machine(2, False, 40, 0, 5, 8, 40)
    g = fstc.compose(m1, m2, small_levels=False)
    assert g.stats["total_product_sources"] == g.num_states - 1
    assert_same(canon_of(g.to_host()), canon_of(oracle.compose(m1, m2)), what="five parts")


@pytest.mark.gpu
@pytest.mark.parametrize("wide", [2000, 2049, 5000])
def test_exact_products_of_long_lists(wide):
    """A state of few parts over thousands of symbols, joined with 12 of them."""
    m1 = machine(1, True, 20, 0, 4, 12, 40, wide=wide, base=wide)
    m2 = machine(2, False, 20, 0, 4, 12, 40, base=wide)
    check(m1, m2, 20)
