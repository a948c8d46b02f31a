"""Prefix reuse, runs of equal bins: requests of a wavefront's length and next
to it, all hits, first accesses at either end of a row, several groups and
weights within a request, few thresholds and more than LDS holds."""
import numpy as np
import pytest

import tracegen as tg
from tests.test_gpu_exclusive import compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("groups,wmax", [(1, 1), (3, 5)])
@pytest.mark.parametrize("caps", [3, 3000])
@pytest.mark.parametrize("length", [1, 63, 64, 65, 128, 200])
def test_request_lengths(oracle_mod, length, caps, groups, wmax):
    rng = np.random.default_rng(length + caps)
    lab, fresh = [], 100_000
    for r in range(60):
        base = 1000 * int(rng.integers(0, 12))
        row = base + np.arange(length)
        cut = int(rng.choice([0, 1, length // 2, length - 1, length]))
        row[cut:] = fresh + np.arange(length - cut)
        fresh += length - cut
        lab.append(row)
    lab = np.concatenate(lab + lab[::3])
    t = tg.from_blocks(lab, weights={int(b): 1 + int(b) % wmax for b in np.unique(lab)},
                       groups={int(b): int(b) // 7 % groups for b in np.unique(lab)}, n_groups=groups, per_request=length)
    c = np.unique(np.linspace(wmax, len(lab) * wmax, caps).astype(int))
    items = [{"cap": (int(a), 0, int(2 * a + 1)), "mode": tg.MODE_INCLUSIVE_PREFIX} for a in c]
    compare(oracle_mod, t, tg.from_list(items), f"prefix-{length}-{caps}-g{groups}-w{wmax}")
