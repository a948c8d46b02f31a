"""Device memory of exclusive evaluations: a batch of FIFO and LFU hierarchies
runs where the trace's load ran (KVCFG_TEST_MEM_CAP, read once per process,
hence a child process).  Counts against the oracle (exact)."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CHILD = r'''
import numpy as np
import tracegen as tg
from oracle import oracle as O
from paper_2603_08739_amd import host
t = tg.random_trace(81, 200_000, 30_000, weight_choices=(1, 4), zipf_s=0.7)
cfgs = tg.from_list([{"cap": (c, d, 900), "policy": p, "mode": tg.MODE_EXCLUSIVE_DEMOTE}
                     for p in (tg.POLICY_FIFO, tg.POLICY_LFU) for c, d in ((300, 4000), (9000, 700))])
h = host.load(t)
counts, _ = host.evaluate(h, cfgs, tg.DEFAULT_COST, 1)
h.free()
np.testing.assert_array_equal(counts, O.replay_memo(t, cfgs))
print("exact")
'''


def test_runs_where_the_load_ran(oracle_mod):
    n, margin = 200_000, 300_000
    # the handle's 20 bytes per access (links, ids, requests, weights, groups)
    # and the load's 24 (hashes, positions, links), request times and counters
    cap = n * (20 + 24) + 8 * n // 4 + margin
    r = subprocess.run([sys.executable, "-c", CHILD], cwd=ROOT, capture_output=True, text=True, timeout=100,
                       env=dict(os.environ, KVCFG_TEST_MEM_CAP=str(cap), PYTHONPATH=ROOT))
    assert r.returncode == 0 and "exact" in r.stdout, r.stderr[-2000:]
