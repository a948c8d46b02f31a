"""kv_trace_load at the limits of its partition bits: a load of 2.3e8 distinct
blocks is linked without the sort that collided hashes take, and traces of
few partition bits (KVCFG_TEST_LOAD_BITS: stretches of thousands of accesses)
give the same results, whether their blocks fit a linking table or not."""
import os

import pytest

from tests.test_gpu_load_partition import check

pytestmark = pytest.mark.gpu


def test_many_distinct_blocks_do_not_sort():
    import torch
    from paper_2603_08739_amd import kvcfg as K
    n = 230_000_000
    i = torch.arange(n, device="cuda")
    req = (i // 100).int()
    h = (i ^ (i >> 5)) * 0x1E3779B97F4A7C15  # injective: an odd multiplier behind a xor-shift
    del i
    K.kv_timing_enable(True)
    try:
        K.kv_timing_read(True)
        t = K.kv_trace_load(h, req, torch.arange(n // 100, device="cuda", dtype=torch.float64))
        calls, _ = K.kv_timing_read(True)["load_sort"]
    finally:
        K.kv_timing_enable(False)
    st = t.info()
    t.free()
    assert (st.n, st.n_distinct, st.max_multiplicity, st.n_w, st.distinct_w) == (n, n, 1, n, n)
    assert calls == 1  # the sort would have been timed under the same name


@pytest.mark.parametrize("bits,n,u", [(1, 20_000, 300), (1, 60_000, 1500), (3, 60_000, 60_000), (5, 70_000, 20_000), (11, 300_000, 200_000)])
def test_few_partition_bits(oracle_mod, bits, n, u):
    os.environ["KVCFG_TEST_LOAD_BITS"] = str(bits)
    try:
        check(oracle_mod, n, u, groups=2, skew=0.3, seed=bits)
    finally:
        os.environ.pop("KVCFG_TEST_LOAD_BITS")
