"""A level of 64 million sources with little to join each: its sources are merged on
the chip in runs that share one set of temp slots (compose.hip, kChunkSlotBytes),
so what the call holds follows the arcs it joins and not the slots that so many
sources would have.  Against the same composition in torch.
"""
import pytest
import torch

from paper_1805_06383_amd import fstc

N = 8000        # states a side; every pair is reached from the start pair
SLOTS = 1 << 34
HUB, FAN = 10, 11  # inner symbols of the hubs and of the start state


def side(hub_arcs, mul, add, seed):
    """(source, target, inner symbol, outer symbol, weight): state 0 leads to
    every state on FAN; state q > 0 has two parallel arcs, on symbols q % 5 and
    q % 5 + 5; every 400th one `hub_arcs` more on HUB, to distinct targets."""
    q = torch.arange(1, N)
    hub = torch.arange(200, N, 400)
    k = torch.arange(hub_arcs).repeat(len(hub))
    hub = hub.repeat_interleave(hub_arcs)
    to = (q * mul + add) % N
    src = torch.cat([torch.zeros(N, dtype=torch.long), q, q, hub])
    dst = torch.cat([torch.arange(N), to, to, (hub + 1 + k) % N])
    inner = torch.cat([torch.full((N,), FAN), q % 5, q % 5 + 5, torch.full_like(hub, HUB)])
    outer = torch.cat([torch.arange(N) % 16, q % 16, q % 16, k % 16])
    g = torch.Generator().manual_seed(seed)
    w = torch.randint(1, 1 << 24, (len(src),), generator=g).float() / (1 << 24)
    order = torch.argsort(src, stable=True)
    return [x[order].cuda() for x in (src, dst, inner, outer, w)]


def device_fst(arcs, inner_is_output):
    src, dst, inner, outer, w = arcs
    il, ol, ni, no = (outer, inner, 16, 12) if inner_is_output else (inner, outer, 12, 16)
    i32 = [x.to(torch.int32) for x in (src, dst, il, ol)]
    return fstc.DeviceFST(N, 0, ni, no, *i32, w, torch.zeros(N, dtype=torch.uint8, device="cuda"))


def arc_key(q1, q2, r1, r2, a, c):
    return ((((q1 * N + q2) * N + r1) * N + r2) * 16 + a) * 16 + c  # 60 bits


def joined(x, y):
    """Sorted arc keys of the composition, their weights and the joined pairs."""
    keys, weights, pairs = [], [], 0
    for sym in range(12):
        i, j = (x[2] == sym).nonzero()[:, 0], (y[2] == sym).nonzero()[:, 0]
        (q1, r1, _, a, w1), (q2, r2, _, c, w2) = ([v[k] for v in s] for s, k in ((x, i), (y, j)))
        k = arc_key(q1[:, None], q2, r1[:, None], r2, a[:, None], c).flatten()
        pairs += k.numel()
        keys.append(k)
        weights.append((w1[:, None] * w2).flatten())
    key, order = torch.cat(keys).sort(stable=True)
    w = torch.cat(weights)[order].double()
    key, n = torch.unique_consecutive(key, return_counts=True)
    last = torch.cumsum(n, 0) - 1
    total = w[last]
    assert int(n.max()) == 2
    two = n == 2
    total[two] += w[last[two] - 1]
    return key, total.float(), pairs


@pytest.mark.gpu
def test_large_sparse_level():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    x, y = side(40, 17, 3, 1), side(10, 13, 1, 2)
    key, weight, pairs = joined(x, y)
    m1, m2 = device_fst(x, True), device_fst(y, False)
    for kw in ({}, dict(deterministic_ids=True), dict(hash_visited=True)):
        r = fstc.fstc_compose(m1, m2, **kw)
        assert (r.num_states, r.num_arcs, r.num_premerge_arcs) == (N * N, key.numel(), pairs)
        # records were written for the start's arcs and the hubs' alone
        assert pairs - r.stats["total_product_records"] == N * N + 20 * 20 * 402
        q = r.state_q1.long() * N + r.state_q2
        if kw.get("deterministic_ids"):
            assert torch.equal(q, torch.arange(N * N, device="cuda"))
        else:
            assert torch.equal(q.sort().values, torch.arange(N * N, device="cuda"))
        src, dst = r.src.long(), r.dst.long()
        assert torch.all(src[1:] >= src[:-1])
        src, dst = q[src], q[dst]
        k = ((src * (N * N) + dst) * 16 + r.ilabel) * 16 + r.olabel
        k, order = k.sort()
        assert torch.equal(k, key)
        # two float32 products and one rounding of their sum, on both sides
        assert torch.equal(r.weight[order], weight)
        # 64 M sources' own slots would take 64e6 * 64 * 17 B; without them the
        # result, the visited set and the start's records are left
        assert r.stats["peak_device_bytes"] < SLOTS + (16 << 30)
        del r, q, src, dst, k, order
