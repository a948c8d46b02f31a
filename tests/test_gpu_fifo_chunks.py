"""FIFO replay: capacities around those at which a job's chunks change length
and thread count (256, 512, 1024 threads for chunks to 1024, 2048, 4096
accesses), blocks of one weight and of several, one group and several, whole
and per-group order, inclusive and exclusive, against the oracle."""
import numpy as np
import pytest

import tracegen as tg
from tests.test_gpu_exclusive import compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("wmax", [1, 7])
@pytest.mark.parametrize("groups,part", [(1, 0), (3, 0), (3, 1)])
@pytest.mark.parametrize("n", [1, 1025, 33_000])
def test_chunk_lengths(oracle_mod, n, groups, part, wmax):
    rng = np.random.default_rng(n + wmax)
    lab = np.where(rng.random(n) < 0.6, rng.zipf(1.1, n) % 20_000, 30_000 + np.arange(n) // 2)
    t = tg.from_blocks(lab, weights={int(b): 1 + int(b) % wmax for b in np.unique(lab)},
                       groups={int(b): int(b) % groups for b in np.unique(lab)}, n_groups=groups, per_request=32)
    items = []
    for c in (63, 64, 1023, 1024, 1087, 1088, 2047, 2048, 2112, 4095, 4096, 9000):
        for m in (0, tg.MODE_EXCLUSIVE_DEMOTE):
            top, low = c * wmax, 3 * c * wmax
            it = {"cap": (top, 0, low), "policy": tg.POLICY_FIFO, "mode": m, "partitioned": part}
            if part:
                it["cap"] = (top * groups, 0, low * groups)
                it["cap_group"] = [[top] * groups, [0] * groups, [low] * groups]
            items.append(it)
    compare(oracle_mod, t, tg.from_list(items), f"fifo-n{n}-g{groups}-p{part}-w{wmax}")
