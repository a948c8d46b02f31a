"""Joint histograms on both sides of the size up to which the stack pass's
first kernel clears them (16,384 words for a trace of one position block),
each evaluated again behind a larger and a smaller batch on the same handle:
what those left behind must not show.  Against the oracle (exact)."""
import numpy as np
import pytest

import tracegen as tg

pytestmark = pytest.mark.gpu


def test_cleared_between_batches(oracle_mod):
    from paper_2603_08739_amd import host
    t = tg.random_trace(511, 900, 120, zipf_s=0.6, reuse_bias=0.2)
    span = float(t.req_time[-1])
    batches = {}
    for caps, ttls in ((5, 3), (63, 62), (63, 64), (100, 200)):  # the second 16,191 words, the third 16,705
        m = max(caps, ttls)
        cfgs = tg.from_list([{"cap": (1 + i % caps, 0, 0), "ttl": span * (i % ttls) / ttls} for i in range(m)])
        batches[caps, ttls] = cfgs, oracle_mod.replay_memo(t, cfgs)
    h = host.load(t)
    for key in [(63, 62), (100, 200), (63, 62), (63, 64), (100, 200), (63, 64), (5, 3), (100, 200), (5, 3)]:
        cfgs, ref = batches[key]
        print("  batch", key, flush=True)
        counts, _ = host.evaluate(h, cfgs, tg.DEFAULT_COST, 1)
        np.testing.assert_array_equal(counts, ref)
    h.free()
