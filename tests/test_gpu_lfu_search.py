"""LFU replay: victims whose class has its oldest member far behind (more
positions than one wavefront searches, so the whole block does), at counts
with and without a head in LDS, with no member before the walked accesses,
and after class 1 ran dry; inclusive and exclusive, against the oracle."""
import numpy as np
import pytest

import tracegen as tg
from tests.test_gpu_exclusive import compare

pytestmark = pytest.mark.gpu


def trace(lead, count, groups, seed):
    """A long lead of hot blocks, then blocks touched `count` times each, the
    hot ones again, and new blocks that have to evict the former."""
    rng = np.random.default_rng(seed)
    hot = np.arange(50)
    warm = np.repeat(np.arange(100, 350), count)
    rng.shuffle(warm)
    again = np.resize(hot, 9000)
    fresh = np.concatenate([np.repeat(np.arange(1000 + 40 * k, 1040 + 40 * k), 1 + k % 3) for k in range(60)])
    lab = np.concatenate([np.resize(hot, lead), warm, again, fresh, np.arange(100, 350), again, fresh[::-1]])
    lab = np.concatenate([lab, lab[lead:] + 5000])
    g = {int(b): int(b) % groups for b in np.unique(lab)}
    return tg.from_blocks(lab, groups=g, n_groups=groups, per_request=16)


@pytest.mark.parametrize("count", [2, 3, 70])
@pytest.mark.parametrize("lead,groups", [(2000, 1), (4160, 1), (40_000, 1), (40_000, 2)])
def test_far_victims(oracle_mod, lead, count, groups):
    t = trace(lead, count, groups, lead + count)
    caps = [(300, 0, 0), (301, 310, 0), (280, 320, 900)]
    items = [{"cap": c, "policy": tg.POLICY_LFU, "mode": m} for c in caps for m in (0, tg.MODE_EXCLUSIVE_DEMOTE)]
    compare(oracle_mod, t, tg.from_list(items), f"far-lead{lead}-count{count}-g{groups}")
