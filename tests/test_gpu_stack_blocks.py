"""The stack pass at every size of its position blocks, forced for short
traces: lengths next to one, two and three blocks, one weight and mixed
weights, shared and partitioned caches, inclusive and write-back-demotion
LRU, prefix reuse, TTL disks and leaf-first eviction, against the oracle."""
import numpy as np
import pytest

import tracegen as tg
from tests.test_gpu_paths import check

pytestmark = pytest.mark.gpu


def batch(t, mixed):
    u, w = int(t.n), int(t.weight.max())
    caps = [(max(w, u // 40), max(w, u // 9), max(w, u)), (w, 0, max(w, u // 3)), (max(w, u // 7), w, 0), (0, max(w, u // 100), 0)]
    items = [{"cap": c} for c in caps] + [{"cap": c, "mode": tg.MODE_INCLUSIVE_PREFIX} for c in caps]
    items += [{"cap": (c[0], c[1], 0), "ttl": [3.0, 40.0, 11.5][: t.n_groups]} for c in caps]
    if not mixed:
        items += [{"cap": c, "mode": tg.MODE_EXCLUSIVE_DEMOTE} for c in caps]
    if t.n_groups > 1:
        for c in caps:
            cg = np.asarray([[max(w, x // t.n_groups) if x else 0] * t.n_groups for x in c], np.uint64)
            items.append({"cap": tuple(int(x) for x in cg.sum(axis=1)), "cap_group": cg, "partitioned": 1})
    return tg.from_list(items)


@pytest.mark.parametrize("weights", [(1,), (3,), (1, 4)])
@pytest.mark.parametrize("logb", [10, 11, 12, 13])
def test_block_edges(oracle_mod, logb, weights):
    b = 1 << logb
    for n, groups in ((1, 1), (b - 1, 1), (b, 2), (b + 1, 3), (2 * b + 5, 2), (3 * b, 1), (4 * b - 1, 2)):
        t = tg.random_trace(n + groups, n, max(2, n // 6), n_groups=groups, weight_choices=weights, zipf_s=0.7)
        check(oracle_mod, t, batch(t, len(weights) > 1), f"block{logb}-n{n}-w{weights}", KVCFG_TEST_BLOCK_LOG=logb)


@pytest.mark.parametrize("logb", [10, 12])
def test_leaf_order(oracle_mod, logb):
    t = tg.tiny(n_req=60)
    c = tg.from_list([{"cap": (k, 2 * k, 0), "policy": tg.POLICY_LEAF} for k in (1500, 2500, 4000)])
    check(oracle_mod, t, c, f"leaf-block{logb}", KVCFG_TEST_BLOCK_LOG=logb)
