"""moe_trans and moe_agg against plain indexing: hosted experts beyond the first 64, unused slots, tensors of different sizes
in one call (one shorter than a block's trip, one longer than the grid), versions that keep a slot, and tensors of a call
that write to the same pool (taken in the order of the call)."""
import numpy as np
import pytest
import torch

import gpu_util as G
from paper_2411_10003_amd import binding

pytestmark = pytest.mark.gpu


def _handle(E, Gc):
    return binding.Handle(T=64, d=64, h=64, E=E, k=1, P=3, self_dest=1, G=Gc, dtype="bf16", act="gelu", renorm=0, device=G.DEV)


def _dest(E, hosted):
    dest = np.full(E, 2, np.int32)
    dest[: E // 2] = 0
    dest[hosted] = 1
    return G.dev(dest)


@pytest.mark.parametrize("E,hosted,Gc", [(3, [1], 2), (64, [0, 63], 2), (130, [2, 63, 64, 100, 128, 129], 8), (1000, [999], 1), (16, [], 3)])
def test_gather_and_add(E, hosted, Gc):
    rng = torch.Generator(device=G.DEV).manual_seed(E)
    hd, dest = _handle(E, Gc), _dest(E, hosted)
    sizes = [8, 1000 * 8, 70000 if E <= 130 else 8]
    pools = [torch.randn(E, n, generator=rng, device=G.DEV) for n in sizes]
    groups = [torch.full((Gc, n), 7.0, device=G.DEV) for n in sizes]
    slot_expert = torch.full((Gc,), -1, dtype=torch.int32, device=G.DEV)
    slot_version = torch.full((Gc,), -1, dtype=torch.int32, device=G.DEV)
    version = torch.zeros(E, dtype=torch.int32, device=G.DEV)
    hd.trans(dest, slot_expert, pools, groups, version, slot_version)
    for p, q in zip(pools, groups):
        for g in range(Gc):
            assert torch.equal(q[g], p[hosted[g]] if g < len(hosted) else torch.full_like(q[g], 7.0))
    assert G.host(slot_expert).tolist() == hosted + [-1] * (Gc - len(hosted))
    assert G.host(slot_version).tolist() == [0] * len(hosted) + [-1] * (Gc - len(hosted))
    # only the expert with a new version is copied again
    for p in pools:
        p += 1.0
    if hosted:
        version[hosted[-1]] = 5
    before = [q.clone() for q in groups]
    hd.trans(dest, slot_expert, pools, groups, version, slot_version)
    for p, q, b in zip(pools, groups, before):
        for g in range(len(hosted)):
            assert torch.equal(q[g], p[hosted[g]] if g == len(hosted) - 1 else b[g])
    grads = [torch.randn(Gc, n, generator=rng, device=G.DEV) for n in sizes]
    want = [p.clone() for p in pools]
    for w, q in zip(want, grads):
        for g, e in enumerate(hosted):
            w[e] += q[g]
    hd.agg(dest, grads, pools)
    assert all(torch.equal(p, w) for p, w in zip(pools, want))


def test_two_tensors_into_one_pool():
    E, hosted = 20, [3, 7, 19]
    hd, dest = _handle(E, 3), _dest(E, hosted)
    pool = torch.randn(E, 4096, device=G.DEV)
    a, b = torch.randn(3, 4096, device=G.DEV), torch.randn(3, 4096, device=G.DEV)
    want = pool.clone()
    for g, e in enumerate(hosted):
        want[e] = (want[e] + a[g]) + b[g]
    hd.agg(dest, [a, b], [pool, pool])
    assert torch.equal(pool, want)
    other = torch.randn(E, 4096, device=G.DEV)
    groups = torch.zeros(3, 4096, device=G.DEV)
    hd.trans(dest, torch.full((3,), -1, dtype=torch.int32, device=G.DEV), [pool, other], [groups, groups])
    assert torch.equal(groups, other[hosted])


@pytest.mark.parametrize("n", [8388604, 8388608, 8388620])     # two slots: just under 64 MB, at it, and past it with a last short trip
def test_streamed_moves(n):
    E, hosted = 4, [1, 3]
    hd, dest = _handle(E, 2), _dest(E, hosted)
    pool, groups = torch.randn(E, n, device=G.DEV), torch.zeros(2, n, device=G.DEV)
    hd.trans(dest, torch.full((2,), -1, dtype=torch.int32, device=G.DEV), [pool], [groups])
    assert torch.equal(groups, pool[hosted])
    want = pool.clone()
    want[hosted] += groups
    hd.agg(dest, [groups], [pool])
    assert torch.equal(pool, want)
