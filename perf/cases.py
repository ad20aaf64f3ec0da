"""What the speed of this library is measured on: compositions as a program asks for them.

A program holds two transducers on the GPU (their coordinate lists, ``fstc.DeviceFST``) and calls
``fstc.fstc_compose`` or ``fstc.fstc_compose_eps``; it gets the reachable states and the arcs back as
tensors.  There is no plan to keep between calls: the layout of both inputs is built inside each
call, so one pass is the whole of it.

Most cases number the states reproducibly (``deterministic_ids``).  By default the numbering within
a depth is the order in which workgroups reach the pairs and differs from call to call, so a program
that stores a composition, compares two of them or addresses its states later asks for the ordered
ids.  The default numbering is measured by ``hmm-table``, whose program addresses states by their
pair, and by ``pivot``, which has one state.

The inputs are drawn by ``paper_1805_06383_amd.workloads``.  A case fixes their graph up to names, so
that every seed's result has the same size; the seed renames the states and the symbols of all three
alphabets and draws the weights, k / 2**24.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1805_06383_amd import fstc
from paper_1805_06383_amd import workloads as W

# Sizes of a family's inputs, and what else its calls are asked for:
#   random     tiny_random on both sides, the start state a busiest one: |Q|, arcs, inner alphabet
#   lm         bigram language model x translation model on both sides (words of the three tongues)
#   sparse     uniform sources and targets, Zipf inner symbols: |Q|, arcs, inner alphabet, depth cap
#   lexicon    prefix tree of words against a one-state dictionary
#   hmm        every state has an arc for each (outer symbol, target) slot and each inner symbol
#   powerlaw   out-degrees by a power law, a busiest state as start: |Q|, arcs, inner alphabet, cap
#   pivot      two one-state translation tables joined over the words of a middle tongue
#   eps        labels are the empty string with some probability on every tape
FAMILIES = ("random", "lm", "sparse", "lexicon", "hmm", "powerlaw", "pivot", "eps")


def listed():
    return [
        # the smallest: a grammar fragment of a few dozen states, composed once per utterance;
        # launches, waits and the host's own work are all there is
        dict(name="tiny", family="random", states=30, arcs=150, inner=8, ids=True),
        # translation models of a small training set (about 1,400 states, 10,000 arcs come out):
        # a handful of short levels
        dict(name="lm-small", family="lm", words1=3506, words2=4657, words3=3506,
             arcs1=16_500, arcs2=15_400, ids=True),
        # the same at the largest training size: 25,000 states and 158,000 arcs to lay out, about
        # 9,000 states and 80,000 arcs come out
        dict(name="lm-large", family="lm", words1=14_176, words2=25_178, words3=14_176,
             arcs1=158_000, arcs2=126_000, ids=True),
        # two one-state translation tables over a shared middle vocabulary: one source state whose
        # millions of joined arcs are merged by (input word, output word)
        dict(name="pivot", family="pivot", words1=20_000, words2=15_000, words3=20_000,
             arcs1=60_000, arcs2=60_000),
        # sparse transducers with a wide inner alphabet: millions of states with about eight joined
        # arcs each, hardly any of them merged
        dict(name="sparse", family="sparse", states=10_000, arcs=200_000, inner=5_000, outer=2_000,
             levels=9, ids=True),
        # a dictionary: 250,000 trie nodes against one state with 150,000 loops
        dict(name="lexicon", family="lexicon", words=50_000, chars=30, out=20_000, ids=True),
        # dense inner alphabet, 64 joined arcs merged into each of the result's: the workload the
        # repository quotes its throughput on, addressed by state pair
        dict(name="hmm-table", family="hmm", states=1000, inner=64, outer=64, slots=4),
        # the same with reproducible ids
        dict(name="hmm", family="hmm", states=1000, inner=64, outer=64, slots=4, ids=True),
        # ten slots a state, more than the matrix form takes: 1,600 joined arcs a source go through
        # written records
        dict(name="hmm-wide", family="hmm", states=200, inner=16, outer=64, slots=10, ids=True),
        # without reduction (every joined arc kept): what a program asks for that sums elsewhere
        dict(name="hmm-unreduced", family="hmm", states=250, inner=64, outer=64, slots=4, ids=True,
             reduce=False),
        # hubs: a start state with thousands of arcs and a visited set in the hash table
        dict(name="powerlaw", family="powerlaw", states=100_000, arcs=2_000_000, inner=20_000,
             outer=5_000, dmax=4_000, levels=2, ids=True),
        # empty strings on all four tapes (three-state filter, two compositions in one call)
        dict(name="eps", family="eps", states=2000, arcs=40_000, inner=1000, outer=500, ids=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of one of the families, sizes over its range and no case above the largest listed."""
    return dict(_draw(rng), graph=rng.randint(1, 10**6))


def _draw(rng):
    family = rng.choice(FAMILIES)
    ids = rng.random() < 0.75
    if family == "random":
        n = _log(rng, 12, 120)
        return dict(family=family, states=n, arcs=5 * n, inner=rng.randint(6, 9), ids=True)
    if family == "lm":
        v = _log(rng, 1500, 20_000)
        a = int(v * rng.uniform(4.5, 7.0))
        return dict(family=family, words1=int(v * rng.uniform(0.6, 1.0)), words2=v,
                    words3=int(v * rng.uniform(0.6, 1.0)), arcs1=a,
                    arcs2=int(a * rng.uniform(0.8, 1.0)), ids=True)
    if family == "sparse":
        n = _log(rng, 3000, 20_000)
        return dict(family=family, states=n, arcs=int(n * rng.uniform(16, 22)),
                    inner=rng.randint(4000, 6000), outer=_log(rng, 200, 5000),
                    levels=rng.randint(5, 8), ids=True)
    if family == "lexicon":
        return dict(family=family, words=_log(rng, 3000, 50_000), chars=rng.randint(20, 40),
                    out=_log(rng, 2000, 20_000), ids=True)
    if family == "hmm":
        slots = rng.randint(2, 11)
        inner = rng.randint(8, 64) if slots <= 4 else rng.randint(8, max(8, min(64, 1600 // slots**2)))
        n = _log(rng, 60, min(1000, int(2000 / slots)))
        reduce = rng.random() < 0.8
        if not reduce:
            n = min(n, int(math.sqrt(4_000_000_000 / 64 / (inner * slots * slots))))
        return dict(family=family, states=n, inner=inner, outer=rng.randint(20, 70), slots=slots,
                    ids=ids or not reduce, reduce=reduce)
    if family == "powerlaw":
        n = _log(rng, 10_000, 100_000)
        return dict(family=family, states=n, arcs=int(n * rng.uniform(12, 20)), inner=n // 5,
                    outer=rng.randint(1000, 5000), dmax=max(400, n // 25), levels=2, ids=True)
    if family == "pivot":
        v = _log(rng, 500, 20_000)
        return dict(family=family, words1=v, words2=int(v * rng.uniform(0.5, 1.0)),
                    words3=int(v * rng.uniform(0.5, 1.0)), arcs1=int(v * rng.uniform(2, 3)),
                    arcs2=int(v * rng.uniform(2, 3)), ids=ids)
    n = _log(rng, 200, 2000)
    return dict(family=family, states=n, arcs=20 * n, inner=n // 2, outer=rng.randint(50, 500),
                ids=True)


def _table(rng, nin, nout, arcs):
    """One state with `arcs` loops: input words by Zipf(0.7), output words by Zipf(0.7)."""
    z = np.zeros(arcs)
    return W.FST(1, 0, nin, nout, z, z, W._zipf(rng, nin, 0.7, arcs), W._zipf(rng, nout, 0.7, arcs),
                 W.random_weights(rng, arcs), np.ones(1, dtype=np.uint8))


def _busiest_start(m):
    m.start = int(np.argmax(np.bincount(m.src, minlength=m.num_states)))
    return m


def _graph(case):
    """The two transducers of a case on the host, up to names and weights."""
    family, seed = case["family"], case.get("graph", 0)
    rng = np.random.default_rng(seed)
    if family == "random":
        n, a, g = case["states"], case["arcs"], case["inner"]
        return (_busiest_start(W.tiny_random(rng, n, 20, g, a)),
                _busiest_start(W.tiny_random(rng, n, g, 20, a)))
    if family == "lm":
        return (W.lm_tm(rng, case["words1"], case["words2"], case["arcs1"]),
                W.lm_tm(rng, case["words2"], case["words3"], case["arcs2"]))
    if family == "sparse":
        n, a, g, o = case["states"], case["arcs"], case["inner"], case["outer"]

        def one(inner_is_output):
            src, dst = rng.integers(0, n, a), rng.integers(0, n, a)
            inner, outer = W._zipf(rng, g, 1.0, a), rng.integers(0, o, a)
            il, ol, nin, nout = (outer, inner, o, g) if inner_is_output else (inner, outer, g, o)
            return W.FST(n, 0, nin, nout, src, dst, il, ol, W.random_weights(rng, a),
                         (rng.random(n) < 0.05).astype(np.uint8))
        return one(True), one(False)
    if family == "lexicon":
        return W.config3(seed, num_words=case["words"], num_chars=case["chars"], num_out=case["out"])
    if family == "hmm":
        return W.config4(seed, nq=case["states"], m=case["inner"], nsym=case["outer"],
                         slots=case["slots"])
    if family == "powerlaw":
        return W.config5(seed, nq=case["states"], na=case["arcs"], ng=case["inner"],
                         nouter=case["outer"], dmax=case["dmax"])
    if family == "pivot":
        return (_table(rng, case["words1"], case["words2"], case["arcs1"]),
                _table(rng, case["words2"], case["words3"], case["arcs2"]))
    return W.eps_pair(seed, nq=case["states"], narcs=case["arcs"], nsym=case["inner"],
                      nouter=case["outer"], eps_inner=0.05, eps_outer=0.05)


def _renamed(m, rng, states, isyms, osyms):
    """The transducer with its states and symbols renamed and new weights; arcs listed by source
    state stay so."""
    src, dst = states[m.src], states[m.dst]
    il, ol, w = isyms[m.ilabel], osyms[m.olabel], W.random_weights(rng, m.num_arcs)
    if m.num_arcs and np.all(m.src[1:] >= m.src[:-1]):
        order = np.argsort(src, kind="stable")
        src, dst, il, ol = src[order], dst[order], il[order], ol[order]
    final = np.zeros_like(m.final)
    final[states] = m.final
    return W.FST(m.num_states, int(states[m.start]), m.num_isyms, m.num_osyms, src, dst, il, ol, w, final)


def _inputs(case, seed):
    """The two transducers of a case on the host."""
    m1, m2 = _graph(case)
    rng = np.random.default_rng(int(seed) % (1 << 31))
    x, y, z = (rng.permutation(n) for n in (m1.num_isyms, m1.num_osyms, m2.num_osyms))
    if case["family"] == "eps":  # label 0 stays the empty string
        x, y, z = (np.concatenate([[0], 1 + rng.permutation(len(v) - 1)]) for v in (x, y, z))
    return (_renamed(m1, rng, rng.permutation(m1.num_states), x, y),
            _renamed(m2, rng, rng.permutation(m2.num_states), y, z))


def prepare(case, seed):
    m1, m2 = _inputs(case, seed)
    return dict(case=case, m1=fstc.DeviceFST.from_host(m1), m2=fstc.DeviceFST.from_host(m2))


def _compose(state):
    case = state["case"]
    kw = dict(max_levels=case.get("levels", 0), deterministic_ids=bool(case.get("ids", False)),
              reduce=bool(case.get("reduce", True)), want_stats=False)
    if case["family"] == "eps":
        return fstc.fstc_compose_eps(state["m1"], state["m2"], 0, **kw)
    return fstc.fstc_compose(state["m1"], state["m2"], **kw)


def _outputs(r):
    out = dict(q1=r.state_q1, q2=r.state_q2, final=r.final, src=r.src, dst=r.dst, il=r.ilabel,
               ol=r.olabel, weight=r.weight)
    if r.state_filter is not None:
        out["filter"] = r.state_filter
    return out


def _pair_table(q1, q2, src, dst, il, ol, weight, final, n1, n2, slots):
    """The composition as tables over state pairs: row q1 |Q2| + q2 holds the pair's arcs in their
    order (by target and labels), at most slots**2 of them, and whether the pair accepts."""
    row = q1 * n2 + q2
    first = torch.searchsorted(src, torch.arange(q1.numel(), dtype=src.dtype, device=src.device),
                               out_int32=True)
    width = slots * slots
    at = torch.arange(src.numel(), dtype=torch.int32, device=src.device)
    at = ((row * width - first).index_select(0, src) + at).long()
    size = n1 * n2 * width
    out = dict(weight=torch.zeros(size, dtype=weight.dtype, device=src.device),
               to=torch.full((size,), -1, dtype=torch.int32, device=src.device),
               labels=torch.full((size,), -1, dtype=torch.int32, device=src.device),
               final=torch.full((n1 * n2,), -1, dtype=torch.int8, device=src.device))
    out["weight"].scatter_(0, at, weight)
    out["to"].scatter_(0, at, row.index_select(0, dst))
    out["labels"].scatter_(0, at, il * 65536 + ol)
    out["final"].scatter_(0, row.long(), final.to(torch.int8))
    return out


def run(state):
    case = state["case"]
    r = _compose(state)
    if case["family"] == "hmm" and not case.get("ids", False):
        return _pair_table(r.state_q1, r.state_q2, r.src, r.dst, r.ilabel, r.olabel, r.weight, r.final,
                           state["m1"].num_states, state["m2"].num_states, case["slots"])
    return _outputs(r)


def work(case):
    """Both inputs read once (20 B an arc, 1 B a state), the result written once (20 B an arc, 9 B a
    state); a multiplication and an addition for each joined arc pair.  How much of the graph can be
    reached is the same for every seed and is taken from a composition."""
    state = prepare(case, 1)
    r = _compose(state)
    n = 20 * (state["m1"].num_arcs + state["m2"].num_arcs) + state["m1"].num_states + state["m2"].num_states
    return dict(bytes=n + 20 * r.num_arcs + 9 * r.num_states, flops=2 * r.num_premerge_arcs)


def tolerance(case):
    """Weights are sums of 32-bit products held in 64 bits and rounded to 32 bits once.  Against
    64-bit products and sums every family is 1e-8 to 3e-8 off: four times that, and two units in the
    last place for the single worst weight.  Ids, labels and flags are exact."""
    return dict(rel=1.2e-7, max=2.4e-7)


# ---------------------------------------------------------------------------------------------
# The same composition in plain torch: breadth-first over state pairs, the joined arcs of a level
# by search in the other side's arcs sorted by (state, inner symbol), products and sums in 64 bits.

class _Side:
    """Arcs of one transducer sorted by (state, inner symbol), then by the rank of their
    (state, target, outer symbol), then as given."""

    def __init__(self, n, nsym, src, dst, inner, outer, weight):
        nout = int(outer.max()) + 1 if outer.numel() else 1
        part = (src * n + dst) * nout + outer
        self.parts, rank = torch.unique(part, return_inverse=True)
        self.target, self.outer = (self.parts // nout) % n, self.parts % nout
        order = torch.argsort(rank, stable=True)
        key = src * nsym + inner
        order = order[torch.argsort(key[order], stable=True)]
        self.nsym, self.key, self.rank = nsym, key[order], rank[order]
        self.inner, self.weight = inner[order], weight[order].double()
        states = torch.arange(n + 1, device=src.device)
        self.row = torch.searchsorted(src[order].contiguous(), states)
        self.max_degree = int((self.row[1:] - self.row[:-1]).max()) if n else 0


def _spread(count):
    """(index of the group, place within it) of every element of groups of these sizes."""
    group = torch.repeat_interleave(torch.arange(count.numel(), device=count.device), count)
    first = torch.cumsum(count, 0) - count
    return group, torch.arange(group.numel(), device=count.device) - first[group]


def _expand(a, b, q1, q2, reduce, most=1 << 26):
    """Arcs of the sources (q1[i], q2[i]): source, M1 part, M2 part, weight, and the joined pairs.
    Without reduction they come by source, symbol, M1 arc, M2 arc, else by source and parts."""
    degree = a.row[q1 + 1] - a.row[q1]
    got, pairs, lo = [], 0, 0
    n = q1.numel()
    total = torch.cumsum(degree, 0)
    while lo < n:  # as many sources at once as keep the pairs in memory
        hi = lo + max(1, int(torch.searchsorted(total, int(total[lo - 1] if lo else 0) + most // 16)) - lo)
        u, k = _spread(degree[lo:hi])
        u += lo
        i = a.row[q1[u]] + k
        want = q2[u] * b.nsym + a.inner[i]
        first = torch.searchsorted(b.key, want)
        count = torch.searchsorted(b.key, want, right=True) - first
        g, k = _spread(count)
        j = first[g] + k
        pairs += j.numel()
        su, p1, p2 = u[g], a.rank[i[g]], b.rank[j]
        w = a.weight[i[g]] * b.weight[j]
        if reduce and j.numel():
            n1, n2 = a.parts.numel(), b.parts.numel()
            key = ((su - lo) * n1 + p1) * n2 + p2
            key, at = torch.unique(key, return_inverse=True)
            w = torch.zeros(key.numel(), dtype=torch.float64, device=w.device).index_add_(0, at, w)
            su, p1, p2 = key // (n1 * n2) + lo, key // n2 % n1, key % n2
        got.append((su, p1, p2, w))
        lo = hi
    return [torch.cat(x) for x in zip(*got)], pairs


def _reference(a, b, f1, f2, start1, start2, levels, reduce):
    """States in breadth-first order, by (q1, q2) within a depth, and their arcs."""
    dev = f1.device
    n2 = f2.numel()
    known = torch.tensor([start1 * n2 + start2], device=dev)  # sorted pairs and their ids
    ids = torch.zeros(1, dtype=torch.long, device=dev)
    frontier, states, arcs, depth, base = known, [known], [], 0, 0
    while frontier.numel() and (not levels or depth < levels):
        (u, p1, p2, w), pairs = _expand(a, b, frontier // n2, frontier % n2, reduce)
        if not pairs:
            break
        to = a.target[p1] * n2 + b.target[p2]
        fresh = torch.unique(to)
        at = torch.searchsorted(known, fresh).clamp_(max=known.numel() - 1)
        fresh = fresh[known[at] != fresh]
        next_base = base + frontier.numel()
        known, order = torch.sort(torch.cat([known, fresh]))
        ids = torch.cat([ids, next_base + torch.arange(fresh.numel(), device=dev)])[order]
        arcs.append((base + u, to, a.outer[p1], b.outer[p2], w))
        states.append(fresh)
        frontier, base, depth = fresh, next_base, depth + 1
    states = torch.cat(states)
    if arcs:
        src, to, il, ol, w = (torch.cat(x) for x in zip(*arcs))
    else:
        src = to = il = ol = torch.zeros(0, dtype=torch.long, device=dev)
        w = torch.zeros(0, dtype=torch.float64, device=dev)
    dst = ids[torch.searchsorted(known, to)]
    q1, q2 = states // n2, states % n2
    return dict(q1=q1, q2=q2, final=((f1[q1] != 0) & (f2[q2] != 0)).to(torch.uint8), src=src, dst=dst,
                il=il, ol=ol, weight=w)


def _eps_reference(x, y, nsym, levels, reduce, dev):
    """Label 0 is the empty string: M1's empty outputs become symbol E2 (M1 moves alone, or with M2)
    and its states loop on E1; M2's empty inputs become E1 and its states loop on E2; the filter
    state is the one of the published three-state epsilon filter."""
    e1, e2 = nsym, nsym + 1

    def loops(m, inner, outer, empty, loop):
        n = m["n"]
        q = torch.arange(n, device=dev)
        o = torch.zeros_like(q)
        return dict(n=n, src=torch.cat([m["src"], q]), dst=torch.cat([m["dst"], q]),
                    inner=torch.cat([torch.where(inner == 0, empty, inner), o + loop]),
                    outer=torch.cat([outer, o]), w=torch.cat([m["w"], torch.ones(n, dtype=torch.float64, device=dev)]),
                    f=m["f"], start=m["start"])
    a = loops(x, x["ol"], x["il"], e2, e1)
    b = loops(y, y["il"], y["ol"], e1, e2)
    # the filter: (state, read from M1, written for M2, state)
    sym = torch.arange(1, nsym, device=dev)
    t = [(f, s, s, 0) for f in range(3) for s in sym.tolist()]
    t += [(0, e2, e1, 0), (0, e2, e2, 2), (2, e2, e2, 2), (0, e1, e1, 1), (1, e1, e1, 1)]
    fs, fi, fo, fd = (torch.tensor(v, device=dev) for v in zip(*t))
    # M1' o filter keeps M1's outer label and writes the filter's symbol: a composition whose part
    # is (target, symbol), numbered as a composition without merging is
    sa = _Side(a["n"], nsym + 2, a["src"], a["dst"], a["inner"], a["outer"], a["w"])
    sf = _Side(3, nsym + 2, fs, fd, fi, fo, torch.ones(fs.numel(), device=dev))
    ones = torch.ones(3, dtype=torch.uint8, device=dev)
    m = _reference(sa, sf, a["f"], ones, a["start"], 0, 0, False)
    sm = _Side(m["q1"].numel(), nsym + 2, m["src"], m["dst"], m["ol"], m["il"], m["weight"])
    sb = _Side(b["n"], nsym + 2, b["src"], b["dst"], b["inner"], b["outer"], b["w"])
    r = _reference(sm, sb, m["final"], b["f"], 0, b["start"], levels, reduce)
    r["filter"] = m["q2"][r["q1"]].to(torch.uint8)
    r["q1"] = m["q1"][r["q1"]]
    return r


def exact(case, seed):
    dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
    m1, m2 = _inputs(case, seed)

    def side(m):
        def t(v):
            return torch.from_numpy(np.asarray(v).astype(np.int64)).to(dev)
        return dict(n=m.num_states, start=m.start, src=t(m.src), dst=t(m.dst), il=t(m.ilabel),
                    ol=t(m.olabel), w=torch.from_numpy(m.weight.astype(np.float64)).to(dev),
                    f=torch.from_numpy(m.final).to(dev))
    x, y = side(m1), side(m2)
    levels, reduce = case.get("levels", 0), bool(case.get("reduce", True))
    if case["family"] == "eps":
        r = _eps_reference(x, y, m1.num_osyms, levels, reduce, dev)
    else:
        g = m1.num_osyms
        r = _reference(_Side(x["n"], g, x["src"], x["dst"], x["ol"], x["il"], x["w"]),
                       _Side(y["n"], g, y["src"], y["dst"], y["il"], y["ol"], y["w"]),
                       x["f"], y["f"], x["start"], y["start"], levels, reduce)
    if case["family"] == "hmm" and not case.get("ids", False):
        i = {k: v.to(torch.int32) for k, v in r.items() if k not in ("weight", "final")}
        return _pair_table(i["q1"], i["q2"], i["src"], i["dst"], i["il"], i["ol"], r["weight"],
                           r["final"], x["n"], y["n"], case["slots"])
    small = {k: v.to(torch.int32) for k, v in r.items() if k not in ("weight", "final", "filter")}
    return dict(r, **small)
