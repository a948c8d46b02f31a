"""A call's tables on their way to the device: batches below and above the
sizes that go through pinned memory, several in flight on one trace, and
threads with a trace and a stream each, all against the oracle."""
import threading

import numpy as np
import pytest
import torch

import tracegen as tg
from paper_2603_08739_amd import host, kvcfg

pytestmark = pytest.mark.gpu
PIN = (1 << 20) // 560  # configurations of the largest batch through pinned memory (the smallest: 34 or so)


def batch(n, seed):
    caps = np.cumsum(np.random.default_rng(seed).integers(1, 200, (n, 3)), axis=1)
    return tg.from_list([{"cap": [int(x) for x in c]} for c in caps])


def trace(seed):
    return tg.from_blocks(np.random.default_rng(seed).zipf(1.2, 3000) % 700, per_request=8)


def in_flight(h, batches, stream=None):
    """The batches' counts, all calls made before any is waited for."""
    outs = []
    for b in batches:
        arr, n = host.config_array(b)
        outs.append(torch.zeros((n, 1, 3, 8), dtype=torch.int64, device="cuda"))
        torch.cuda.current_stream().synchronize()  # (zeroed before another stream writes)
        kvcfg.kv_eval_configs(h, arr, n, host.cost_model(tg.DEFAULT_COST), outs[-1], stream=stream)
        del arr
    torch.cuda.synchronize()
    return [o.cpu().numpy().view(np.uint64) for o in outs]


@pytest.mark.parametrize("n", [1, 7, 30, 36, 40, PIN - 40, PIN + 40])
def test_calls_in_flight(oracle_mod, n):
    t = trace(n)
    h = host.load(t)
    batches = [batch(n, s) for s in range(5)]
    for b, got in zip(batches, in_flight(h, batches)):
        np.testing.assert_array_equal(got, oracle_mod.replay(t, b))
    h.free()


def test_threads(oracle_mod):
    out = {}

    def run(i):
        t, st = trace(i), torch.cuda.Stream()
        res = []
        for rep in range(4):
            h = host.load(t, stream=st)
            batches = [batch(30 + i, 10 * i + rep), batch(700 + i, i)]
            res += list(zip(batches, in_flight(h, batches, st)))
            h.free()
        out[i] = (t, res)

    torch.cuda.synchronize()
    ts = [threading.Thread(target=run, args=(i,)) for i in range(4)]
    for x in ts:
        x.start()
    for x in ts:
        x.join()
    assert len(out) == 4
    for t, res in out.values():
        for b, got in res:
            np.testing.assert_array_equal(got, oracle_mod.replay(t, b))
