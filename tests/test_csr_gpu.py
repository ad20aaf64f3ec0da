"""fstc_build_csr on the GPU against a numpy statement of the layout (the
(state, inner symbol) grouping of section 3.3 with per-state part ranks):

* parts: the distinct (state, target, outer symbol) triples in increasing
  order; part_base[q] is the first part of state q, and an arc's part is the
  rank of its (target, outer) among its state's parts;
* segments: the distinct (state, inner symbol) pairs in increasing order;
  row[q] is the first segment of state q; arcs are ordered by (state, inner
  symbol, part, input position), seg_off[k] is the first arc of segment k.

The shapes cover both builds of the library (the per-state build for
transducers with moderate arcs per state, the global sorts otherwise), the
size classes of the per-state build (states of at most 16, 64, 256, 1024
arcs, of more, and of more than one 8192-arc tile) and degenerate symbol
ranges.
"""
import numpy as np
import pytest

from paper_1805_06383_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fstc():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1805_06383_amd import fstc as F
    F.load_library()
    return F


def csr_ref(m, by_output):
    n, nq = m.num_arcs, m.num_states
    src = m.src.astype(np.int64)
    inner = (m.olabel if by_output else m.ilabel).astype(np.int64)
    outer = (m.ilabel if by_output else m.olabel).astype(np.int64)
    trip = np.stack([src, m.dst.astype(np.int64), outer], axis=1)
    uniq, inv = np.unique(trip, axis=0, return_inverse=True)
    inv = inv.reshape(-1)
    part_base = np.searchsorted(uniq[:, 0], np.arange(nq + 1)).astype(np.int64)
    arc_part = inv - part_base[src]
    order = np.lexsort((np.arange(n), arc_part, inner, src))
    pairs = np.stack([src[order], inner[order]], axis=1)
    head = np.ones(n, bool)
    head[1:] = np.any(pairs[1:] != pairs[:-1], axis=1)
    seg_pos = np.flatnonzero(head)
    seg_state = src[order][seg_pos]
    return {
        "row": np.searchsorted(seg_state, np.arange(nq + 1)),
        "seg_sym": inner[order][seg_pos],
        "seg_off": np.append(seg_pos, n),
        "arc_part": arc_part[order],
        "arc_weight": m.weight[order],
        "part_base": part_base,
        "part_target": uniq[:, 1],
        "part_outer": uniq[:, 2],
        "max_parts": int(np.diff(part_base).max()) if nq else 0,
    }


def check(F, m, what):
    for by_out in (True, False):
        c = F.fstc_build_csr(F.DeviceFST.from_host(m), by_out)
        ref = csr_ref(m, by_out)
        S, P = c["num_segments"], c["num_parts"]
        assert S == len(ref["seg_sym"]) and P == len(ref["part_target"]), what
        assert c["max_parts"] == ref["max_parts"], what
        got = {k: c[k].cpu().numpy() for k in ("row", "seg_sym", "seg_off", "arc_part",
                                               "arc_weight", "part_base", "part_target",
                                               "part_outer")}
        n = m.num_arcs
        sizes = {"row": m.num_states + 1, "seg_sym": S, "seg_off": S + 1, "arc_part": n,
                 "arc_weight": n, "part_base": m.num_states + 1, "part_target": P, "part_outer": P}
        for k, ln in sizes.items():
            a = got[k][:ln]
            b = ref[k]
            if k == "arc_weight":
                assert np.array_equal(a.view(np.uint32), b.view(np.uint32)), f"{what} {by_out} {k}"
            else:
                assert np.array_equal(a.astype(np.int64), np.asarray(b, np.int64)), \
                    f"{what} by_output={by_out}: {k} differs"


def skewed(seed, nq, big_state, big_arcs, small_arcs, nin=300, nout=200):
    """States of about small_arcs arcs each, one state with big_arcs."""
    rng = np.random.default_rng(seed)
    src = np.concatenate([rng.integers(0, nq, small_arcs * nq), np.full(big_arcs, big_state)])
    rng.shuffle(src)
    k = len(src)
    return W.FST(num_states=nq, start=0, num_isyms=nin, num_osyms=nout, src=src,
                 dst=rng.integers(0, nq, k), ilabel=rng.integers(0, nin, k),
                 olabel=rng.integers(0, nout, k), weight=W.random_weights(rng, k),
                 final=np.zeros(nq, np.uint8))


@pytest.mark.parametrize("seed", range(6))
def test_csr_tiny(fstc, seed):
    rng = np.random.default_rng(seed)
    m = W.tiny_random(rng, int(rng.integers(1, 9)), int(rng.integers(1, 6)),
                      int(rng.integers(1, 6)), int(rng.integers(1, 60)))
    check(fstc, m, f"tiny {seed}")


@pytest.mark.parametrize("name", ["config1", "config4", "paper1k"])
def test_csr_workloads(fstc, name):
    m1, m2 = {"config1": lambda: W.config1(0), "config4": lambda: W.config4(0),
              "paper1k": lambda: W.paper_pair("1k", "de")}[name]()
    check(fstc, m1, name + " M1")
    check(fstc, m2, name + " M2")


@pytest.mark.parametrize("big", [15, 16, 17, 63, 64, 65, 255, 256, 257, 1023, 1024, 1025, 8191,
                                 8192, 8193, 10_000, 30_001])
def test_csr_state_sizes(fstc, big):
    """One state of `big` arcs among small ones: the size classes and the
    multi-tile sort of the per-state build."""
    check(fstc, skewed(big, 100, 7, big, 10), f"big state {big}")


def test_csr_duplicates_and_degenerate_symbols(fstc):
    rng = np.random.default_rng(5)
    for nin, nout in ((1, 1), (1, 50), (50, 1)):
        m = skewed(nin * 100 + nout, 40, 3, 600, 20, nin, nout)
        m.src[:50] = 3  # some repeated arcs
        m.dst[:50] = 1
        m.ilabel[:50] = 0
        m.olabel[:50] = 0
        check(fstc, m, f"symbols {nin} x {nout}")


def test_csr_global_build(fstc):
    """Shapes that take the global sorts: one state holding most arcs, and
    more states than the per-state build takes."""
    rng = np.random.default_rng(9)
    n = 150_000
    one = W.FST(num_states=1, start=0, num_isyms=5000, num_osyms=3000,
                src=np.zeros(n, np.uint32), dst=np.zeros(n, np.uint32),
                ilabel=rng.integers(0, 5000, n), olabel=rng.integers(0, 3000, n),
                weight=W.random_weights(rng, n), final=np.ones(1, np.uint8))
    check(fstc, one, "one state, 150k arcs")
    many = skewed(3, 200_000, 11, 3000, 2)
    check(fstc, many, "200k states")
    one_small = W.FST(num_states=1, start=0, num_isyms=70, num_osyms=90,
                      src=np.zeros(5000, np.uint32), dst=np.zeros(5000, np.uint32),
                      ilabel=rng.integers(0, 70, 5000), olabel=rng.integers(0, 90, 5000),
                      weight=W.random_weights(rng, 5000), final=np.ones(1, np.uint8))
    check(fstc, one_small, "one state, 5000 arcs")


@pytest.mark.parametrize("nq", [1, 200, 1000, 70_000])
def test_csr_grouped_by_state(fstc, nq):
    """Arcs already grouped by source state (as FST files store them): the
    key pass finds them in order and the state sort's passes (none, one, two
    or three 8-bit passes for these state counts) leave them as they are;
    with one arc out of place the sort runs in full."""
    m = skewed(nq, nq, 0, 40, 3)
    order = np.argsort(m.src, kind="stable")
    for k in ("src", "dst", "ilabel", "olabel", "weight"):
        setattr(m, k, getattr(m, k)[order])
    check(fstc, m, f"grouped, {nq} states")
    m.src[0], m.src[-1] = m.src[-1], m.src[0]
    check(fstc, m, f"grouped, {nq} states, one arc out of place")


@pytest.mark.parametrize("nq,n", [(1, 8192), (1, 8193), (2, 16_384), (2, 16_385), (7, 57_345),
                                  (1, 65_536), (1, 65_537), (1, 16_384), (1, 16_385),
                                  (3, 49_152), (3, 49_153)])
def test_csr_few_large_states(fstc, nq, n):
    """Around the line between the per-state build and the global sorts for
    few states (16,384 arcs on average), and where the former's states take one
    tile of 8,192 arcs or two."""
    rng = np.random.default_rng(n)
    m = W.FST(num_states=nq, start=0, num_isyms=900, num_osyms=1200,
              src=rng.integers(0, nq, n), dst=rng.integers(0, nq, n),
              ilabel=rng.integers(0, 900, n), olabel=rng.integers(0, 1200, n),
              weight=W.random_weights(rng, n), final=np.ones(nq, np.uint8))
    check(fstc, m, f"{nq} states, {n} arcs")


@pytest.mark.parametrize("syms", [2047, 2048, 2049])
def test_long_lists_against_short(fstc, syms):
    """States of few parts and long symbol lists, which the product merge takes
    however long they are, composed with states of 8, 64 and 2,000 symbols."""
    import oracle
    from fstcheck import assert_same, canon_of
    rng = np.random.default_rng(syms)
    src = np.repeat(np.arange(3), syms)
    m1 = W.FST(num_states=3, start=0, num_isyms=4, num_osyms=syms, src=src, dst=(src + 1) % 3,
               ilabel=src % 4, olabel=np.tile(np.arange(syms), 3),
               weight=W.random_weights(rng, 3 * syms), final=np.ones(3, np.uint8))
    k = [8, 2000, 64]
    s2 = np.repeat(np.arange(3), k)
    b2 = np.concatenate([np.sort(rng.choice(syms, x, replace=False)) for x in k])
    m2 = W.FST(num_states=3, start=0, num_isyms=syms, num_osyms=4, src=s2, dst=(s2 + 1) % 3,
               ilabel=b2, olabel=s2 % 4, weight=W.random_weights(rng, len(s2)),
               final=np.ones(3, np.uint8))
    g = fstc.compose(m1, m2, small_levels=False)
    assert_same(canon_of(g.to_host()), canon_of(oracle.compose(m1, m2)), rtol=1e-5, what=f"{syms}")
    assert g.stats["total_product_sources"] > 0
