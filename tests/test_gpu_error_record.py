"""The report of a failed replay names the failing job whatever calls came
after the one that failed, and for the top tiers of exclusive hierarchies too.
(KVCFG_TEST_FAIL_JOB marks a job as failed; every kernel still completes.)"""
import pytest

import tracegen as tg
from tests.test_gpu_paths import env

pytestmark = pytest.mark.gpu


def reported(handle):
    from paper_2603_08739_amd import kvcfg as K
    with pytest.raises(K.KvError) as e:
        handle.info()
    assert e.value.status == K.KV_ERR_DEVICE
    handle.info()  # reported once
    return str(e.value)


def lfu(caps, **kw):
    return tg.from_list([{"cap": (c, d, 0), "policy": tg.POLICY_LFU, **kw} for c, d in caps])


def test_exclusive_top_tier(oracle_mod):
    from paper_2603_08739_amd import host
    t = tg.random_trace(71, 5000, 800, zipf_s=0.8)
    cfgs = tg.ConfigBatch.concat([lfu([(16, 0), (64, 0)]), lfu([(20, 30), (50, 9), (200, 40)], mode=tg.MODE_EXCLUSIVE_DEMOTE)])
    h = host.load(t)
    for job, cap in ((1, 64), (2, 20), (3, 50), (4, 200)):
        with env(KVCFG_TEST_FAIL_JOB=job):
            host.evaluate(h, cfgs, tg.DEFAULT_COST, 1)
        msg = reported(h)
        assert f"replay job {job} (LFU, capacity {cap} granules, shared)" in msg, msg
    counts, _ = host.evaluate(h, cfgs, tg.DEFAULT_COST, 1)
    h.info()
    h.free()
    assert (counts == oracle_mod.replay_memo(t, cfgs)).all()


@pytest.mark.parametrize("after", ["lru", "exclusive", "lfu"])
def test_calls_behind_a_failure(after):
    """The later call is enqueued while the failing one still runs."""
    import torch
    from paper_2603_08739_amd import host, kvcfg as K
    t = tg.random_trace(72, 3_000_000, 400_000, zipf_s=0.7)  # some 10 ms of replay
    first = lfu([(1000 + 37 * i, 0) for i in range(40)])
    later = {"lru": tg.from_list([{"cap": (99, 0, 0)}]), "exclusive": lfu([(7 + i, 50) for i in range(30)], mode=tg.MODE_EXCLUSIVE_DEMOTE),
             "lfu": lfu([(5 + i, 0) for i in range(30)])}[after]
    h = host.load(t)
    model = host.cost_model(tg.DEFAULT_COST)
    arrays = [(host.config_array(c), torch.empty((c.n, 1, 3, 8), dtype=torch.int64, device="cuda")) for c in (first, later)]
    for (a, n), counts in arrays:  # memory is there before
        K.kv_eval_configs(h, a, n, model, counts)
    h.info()
    for _ in range(2):
        (a, n), counts = arrays[0]
        with env(KVCFG_TEST_FAIL_JOB=25):
            K.kv_eval_configs(h, a, n, model, counts)
        (a, n), counts = arrays[1]
        for _again in range(2):
            K.kv_eval_configs(h, a, n, model, counts)
        msg = reported(h)
        assert f"replay job 25 (LFU, capacity {1000 + 37 * 25} granules, shared)" in msg, msg
    h.free()
