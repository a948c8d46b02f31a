"""What a loaded trace keeps on the device: block tables of the distinct blocks,
not of the accesses.  Two long traces of few blocks fit a device memory limit
(KVCFG_TEST_MEM_CAP, read once per process, hence a child process) that their
other arrays and the second load nearly fill; the second one's counts stay
right, mixed weights and groups among them."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
N = 40_000_000
CHILD = r"""
import torch
import numpy as np
import tracegen as tg
from paper_2603_08739_amd import host, kvcfg as K
n, u = %d, 50_000
i = torch.arange(n, device="cuda")
b = (i * 7919) %% u                       # a cycle over u blocks: every distance is known
w, g = (1 + (b & 1)).to(torch.uint8), (b %% 3 == 0).to(torch.uint8)
args = (b * 0x1E3779B97F4A7C15, (i // 1000).int(), torch.arange(n // 1000, device="cuda", dtype=torch.float64), g, w, 2)
first = K.kv_trace_load(*args)
second = K.kv_trace_load(*args)
tot = int((1 + (np.arange(u) & 1)).sum())
cfgs = tg.from_list([{"cap": (c, 0, 0), "policy": p} for c in (tot - 1, tot) for p in (tg.POLICY_LRU, tg.POLICY_FIFO)])
for t in (first, second):
    st = t.info()
    assert (st.n_distinct, st.max_multiplicity, st.distinct_w) == (u, n // u, tot)
first.free()
counts, _ = host.evaluate(second, cfgs, tg.DEFAULT_COST, 2)
per = np.bincount(np.arange(u) %% 3 == 0, minlength=2)
for c in range(4):  # a cyclic scan: every access misses one granule short of all blocks, every re-access hits with all
    hit = counts[c, :, 0, K.FIELDS.index("hit")].tolist()
    assert c >= 2 and hit == [int(x) * (n // u - 1) for x in per] or c < 2 and hit == [0, 0], (c, hit)
print("right")
"""


def test_two_handles_of_few_blocks():
    # a handle: 18 bytes per access; a load beside it: 52, digit counts and request times
    cap = N * (18 + 52) + N // 2 + (8 << 20)
    r = subprocess.run([sys.executable, "-c", CHILD % N], cwd=ROOT, capture_output=True, text=True, timeout=100,
                       env=dict(os.environ, KVCFG_TEST_MEM_CAP=str(cap), PYTHONPATH=ROOT))
    assert r.returncode == 0 and "right" in r.stdout, r.stderr[-2000:]
