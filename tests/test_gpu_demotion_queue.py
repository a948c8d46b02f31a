"""Exclusive hierarchies walked as one demotion queue: trace lengths next to
the walk's 64 lanes, steps of 256 events, staged slices of 2,048 events (and
where the last step before a new slice begins) and windows of 1,024 entries
(events are accesses for LRU over mixed weights), capacities from one block (a head passes entries that the same
step takes out) to all but one block, every policy, one to three live tiers,
shared and partitioned, one and more groups, against the oracle (exact)."""
import numpy as np
import pytest

import tracegen as tg
from tests.test_gpu_exclusive import ALL, compare

pytestmark = pytest.mark.gpu


def batch(caps, groups):
    items = []
    for p in ALL:
        for c in caps:
            items.append({"cap": c, "policy": p, "mode": tg.MODE_EXCLUSIVE_DEMOTE})
            if groups > 1 or p == tg.POLICY_LFU:
                cg = np.zeros((3, groups), np.uint64)
                for k in range(3):
                    cg[k] = max(c[k] // groups, 4) if c[k] else 0
                cap = tuple(int(x) for x in cg.sum(axis=1))
                items.append({"cap": cap, "cap_group": cg, "policy": [p, tg.POLICY_FIFO, p][:groups], "partitioned": 1,
                              "mode": tg.MODE_EXCLUSIVE_DEMOTE})
    return tg.from_list(items)


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 127, 255, 256, 257, 511, 513, 1023, 1024, 1025, 1600, 2047, 2048, 2049, 2303, 2305,
                               4097])
@pytest.mark.parametrize("groups,weights", [(1, (1,)), (1, (1, 4)), (2, (1, 2, 3))])
def test_step_edges(oracle_mod, n, groups, weights):
    t = tg.random_trace(n + 7 * groups, n, max(2, n // 5), n_groups=groups, weight_choices=weights, zipf_s=0.5,
                        reuse_bias=0.2)
    w, u = max(weights), int(max(8, n // 5))
    caps = [(w, w, w), (w, 0, 5 * w), (0, 2 * w + 1, 0), (u // 2 + w, w, 0), (u // 4 + w, u // 4 + w, u // 4 + w),
            (u // 8 + w, 0, u), (0, w, u // 2 + w), (4 * u + w, w, w)]
    compare(oracle_mod, t, batch(caps, groups), f"n{n}-g{groups}-w{weights}")


def test_scans_and_cycles(oracle_mod):
    """Cyclic scans evict every block just before its next access: every event
    takes out an entry at or right behind a head."""
    for period, w in ((40, (1,)), (65, (1, 4)), (600, (1, 4))):
        lab = np.concatenate([np.arange(period)] * (5000 // period) + [np.arange(period)[::-1]])
        t = tg.from_blocks(lab, weights=np.resize(np.asarray(w), period), per_request=16)
        tot = int(np.resize(np.asarray(w), period).sum())
        caps = [(tot - d, max(w) * k, 0) for d in (1, max(w), tot // 2) for k in (1, 2, 9)] + [(tot // 3, tot // 3, tot // 3)]
        compare(oracle_mod, t, batch(caps, 1), f"cycle{period}")


@pytest.mark.parametrize("u,n", [(3, 700), (12, 2500), (60, 5000), (125, 2049)])
@pytest.mark.parametrize("groups,weights", [(1, (1,)), (1, (1, 4)), (2, (1, 2, 3))])
def test_short_recurrences(oracle_mod, u, n, groups, weights):
    """Blocks that come back within the few entries of small tiers, now and
    then or all the time: stretches walked event by event, and long steps
    between them."""
    w = max(weights)
    rng = np.random.default_rng([u, n, groups])
    hot = rng.integers(0, u, n)
    calm = np.where(np.arange(n) // 300 % 2, hot, u + np.arange(n) % 700)  # 300 of each in turn
    for kind, lab in (("hot", hot), ("calm", calm)):
        ids = np.unique(lab)
        t = tg.from_blocks(lab, weights={int(b): weights[int(b) % len(weights)] for b in ids},
                           groups={int(b): int(b) % groups for b in ids}, n_groups=groups, per_request=9)
        caps = [(w, w, w), (w, 3 * w, 9 * w), (2 * w, 0, 5 * w), (u // 4 + w, u // 4 + w, u // 4 + w), (0, w, u // 2 + w), (u // 2 + w, w, 4 * w)]
        compare(oracle_mod, t, batch(caps, groups), f"{kind}-u{u}-n{n}-g{groups}-w{weights}")
