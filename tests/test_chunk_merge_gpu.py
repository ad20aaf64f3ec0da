"""Sources joined and merged on the chip (1 to 8 to a wavefront), against the
oracle and against written records.

Algorithm 2 expands, sorts and sums the arcs of every popped pair (Section
3.4).  A source whose shorter symbol list has at most 64 symbols and that joins
at most 256 arc pairs is merged in its wavefront; the others of the level are
left to the general kernels.  The cases sit at those lines and at the
wavefront's capacities: joined pairs per source of 255 to 257 and more, with
all keys equal and all distinct, lists of 63 to 65 symbols, batches of more
than 256 symbols or records, wavefronts with more merged arcs than slots, long
second lists, levels for every number of sources per wavefront, and levels of
which only a few sources are left.
"""
import numpy as np
import pytest

import oracle
from fstcheck import assert_same, canon_of
from paper_1805_06383_amd import workloads as W


def layered(seed, width, spec1, spec2, syms=400, outer=50, distinct=True):
    """Start state 0 leads to `width` states on its own symbol; state q has
    spec[q % len(spec)] = (symbols, arcs per symbol) arcs to random states."""
    rng = np.random.default_rng(seed)
    nq = width + 1

    def one(spec, inner_is_output):
        src, dst, inner, out = [np.zeros(width, int)], [1 + np.arange(width)], \
            [np.full(width, syms)], [rng.integers(0, outer, width)]
        for q in range(1, nq):
            s, k = spec[q % len(spec)]
            # half of the symbols are the first ones, which all states share
            b = np.r_[np.arange((s + 1) // 2),
                      (s + 1) // 2 + rng.permutation(syms - (s + 1) // 2)[: s // 2]]
            n = len(b) * k
            src.append(np.full(n, q)), inner.append(np.repeat(b, k))
            if distinct:
                dst.append(rng.integers(0, nq, n)), out.append(rng.integers(0, outer, n))
            else:
                dst.append(np.full(n, 1 + q % width)), out.append(np.full(n, q % outer))
        src, dst, inner, out = map(np.concatenate, (src, dst, inner, out))
        p = rng.permutation(len(src))
        src, dst, inner, out = src[p], dst[p], inner[p], out[p]
        il, ol, ni, no = (out, inner, outer, syms + 1) if inner_is_output else \
            (inner, out, syms + 1, outer)
        return W.FST(nq, 0, ni, no, src, dst, il, ol, W.random_weights(rng, len(src)),
                     (rng.random(nq) < 0.4).astype(np.uint8))
    return one(spec1, True), one(spec2, False)


SPECS = {
    "few": ([(1, 1), (2, 1), (3, 2), (0, 1)], [(2, 1), (4, 1), (1, 3)]),
    "pairs-256": ([(1, 16), (1, 15), (1, 17)], [(1, 16), (1, 15), (1, 17)]),
    "pairs-many": ([(3, 20), (1, 60), (5, 3)], [(3, 20), (1, 60), (2, 2)]),
    "lists-64": ([(63, 1), (64, 1), (65, 1), (5, 1)], [(64, 1), (65, 1), (200, 1)]),
    "long-second": ([(3, 1), (1, 2)], [(380, 1), (300, 2)]),
    "full-regions": ([(24, 4), (4, 2)], [(24, 4), (26, 3)]),
}
MODES = {"default": {}, "ordered": dict(deterministic_ids=True),
         "hash": dict(deterministic_ids=True, hash_visited=True), "capped": dict(max_arcs=1 << 40),
         "levels": dict(max_levels=2)}


@pytest.mark.gpu
@pytest.mark.parametrize("mode", list(MODES))
@pytest.mark.parametrize("distinct", [True, False])
@pytest.mark.parametrize("name", list(SPECS))
def test_chunk_shapes(name, distinct, mode):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1805_06383_amd import fstc
    s1, s2 = SPECS[name]
    m1, m2 = layered(len(name), 30, s1, s2, distinct=distinct)
    kw = MODES[mode]
    g = fstc.compose(m1, m2, small_levels=False, **kw)
    ref = oracle.compose(m1, m2, max_levels=kw.get("max_levels", 0))
    h = g.to_host()
    assert_same(canon_of(h), canon_of(ref), rtol=1e-5, what=f"{name} {distinct} {mode}")
    assert h.num_premerge == ref.num_premerge
    assert np.all(h.src[1:] >= h.src[:-1])
    if kw.get("deterministic_ids"):  # the arrays of the written records, order included
        k2 = {k: v for k, v in kw.items()}
        y = fstc.compose(m1, m2, product=False, small_levels=False, **k2).to_host()
        for f in ("q1", "q2", "final", "src", "dst", "a", "c"):
            assert np.array_equal(getattr(h, f), getattr(y, f)), f
        np.testing.assert_allclose(h.w, y.w, rtol=2.5e-7)


@pytest.mark.gpu
@pytest.mark.parametrize("width,cap", [(9, 0), (127, 0), (130, 3), (420, 2), (700, 2)])
def test_chunk_level_sizes(width, cap):
    """Levels of 80 to 490,000 sources: every number of sources a workgroup
    takes, visited sets in both forms."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1805_06383_amd import fstc
    m1, m2 = layered(width, width, [(2, 1), (3, 1), (1, 2)], [(3, 1), (2, 1)], syms=40)
    ref = oracle.compose(m1, m2, max_levels=cap)
    for kw in ({}, dict(deterministic_ids=True), dict(hash_visited=True)):
        h = fstc.compose(m1, m2, max_levels=cap, small_levels=False, **kw).to_host()
        assert_same(canon_of(h), canon_of(ref), rtol=1e-5, what=f"{width} {kw}")


BATCHES = {  # levels of 19,600 sources, 8 to a wavefront
    # 8 x 40 to 64 symbols a wavefront
    "elements": ([(40, 1), (64, 1)], [(64, 1), (50, 1)], True),
    # 8 x up to 225 records, nearly all distinct: more than 512 slots
    "records": ([(15, 3), (2, 2), (5, 4)], [(15, 3), (5, 4)], True),
    # the same with few distinct keys
    "repeats": ([(15, 3), (2, 2), (5, 4)], [(15, 3), (5, 4)], False),
    # one source of 400 records left to the tiles
    "one-left": ([(2, 1)] * 139 + [(1, 20)], [(2, 1)] * 139 + [(1, 20)], True),
}


@pytest.mark.gpu
@pytest.mark.parametrize("name", list(BATCHES))
def test_chunk_batches(name):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1805_06383_amd import fstc
    s1, s2, distinct = BATCHES[name]
    m1, m2 = layered(len(name), 140, s1, s2, distinct=distinct)
    ref = oracle.compose(m1, m2, max_levels=2)
    for kw in ({}, dict(deterministic_ids=True), dict(hash_visited=True)):
        h = fstc.compose(m1, m2, max_levels=2, small_levels=False, **kw).to_host()
        assert_same(canon_of(h), canon_of(ref), rtol=1e-5, what=f"{name} {kw}")
        assert h.num_premerge == ref.num_premerge


@pytest.mark.gpu
def test_chunk_special_weights():
    """Infinities, NaN, zeros and subnormal products, summed like records."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1805_06383_amd import fstc
    m1, m2 = layered(5, 30, [(4, 3), (2, 2)], [(4, 2), (3, 3)], distinct=False)
    rng = np.random.default_rng(1)
    for m in (m1, m2):
        k = rng.integers(0, m.num_arcs, 40)
        m.weight[k] = np.resize(np.array([np.inf, -np.inf, np.nan, 0.0, -0.0, 1e-40, -3e38, 1e38],
                                         np.float32), 40)
    h = fstc.compose(m1, m2, small_levels=False).to_host()
    ref = oracle.compose(m1, m2)
    assert_same(canon_of(h), canon_of(ref), rtol=1e-5, what="special weights")
