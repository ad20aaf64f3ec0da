"""New pairs of merge tiles, listed by the waves that insert the tiles' targets,
against the oracle: tiles of few runs (many to a wave), of full windows (a wave's
list of 1,024 claims appended several times) and sources of more records than a
tile takes, in both forms of the visited set and both numberings.
"""
import pytest

import oracle
from fstcheck import assert_same, canon_of
from paper_1805_06383_amd import workloads as W
from test_chunk_merge_gpu import layered

CASES = {
    # 40,000 sources, 64 joined pairs merged into each run
    "few-runs": (lambda: W.config4(3, nq=200, m=64, slots=2), 0),
    # 8,100 sources, hardly any run repeats: new pairs by the thousand
    "full-tiles": (lambda: layered(4, 90, [(15, 3), (2, 2)], [(15, 3), (5, 4)]), 2),
    # one source of 60 x 60 pairs among sparse ones: a tile of its own
    "mid": (lambda: layered(5, 40, [(2, 1)] * 39 + [(1, 60)], [(2, 1)] * 39 + [(1, 60)]), 3),
    "one-run": (lambda: layered(6, 60, [(1, 1)], [(1, 1)]), 0),
}


@pytest.mark.gpu
@pytest.mark.parametrize("mode", [{}, dict(deterministic_ids=True), dict(hash_visited=True),
                                  dict(max_arcs=1 << 40)],
                         ids=["default", "ordered", "hash", "capped"])
@pytest.mark.parametrize("name", list(CASES))
def test_claims_of_tiles(name, mode):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1805_06383_amd import fstc
    make, cap = CASES[name]
    m1, m2 = make()
    h = fstc.compose(m1, m2, max_levels=cap, product=False, small_levels=False, **mode).to_host()
    assert_same(canon_of(h), canon_of(oracle.compose(m1, m2, max_levels=cap)), what=name)
