"""kv_trace_load with far more requests than accesses: every request time is
checked and copied, in a time that does not grow with requests per access."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def load(n, times):
    import torch
    from paper_2603_08739_amd import kvcfg as K
    req = torch.linspace(0, len(times) - 1, n, device="cuda", dtype=torch.float64).int()
    return K.kv_trace_load(torch.arange(n, device="cuda") // 3, req, times)


@pytest.mark.parametrize("n,n_req", [(1, 1), (1, 8193), (1000, 3_000_001), (8193, 20_000_000)])
def test_times_are_checked(n, n_req):
    import torch
    from paper_2603_08739_amd import kvcfg as K
    times = torch.arange(n_req, device="cuda", dtype=torch.float64)
    t = load(n, times)
    assert t.info().span == n_req - 1
    if n > 2:  # the gap between an access and the next of its block is in request times: all were copied
        out = [torch.empty((1, 3), dtype=d, device="cuda") for d in (torch.int64, torch.int64, torch.float64)]
        gaps = np.diff(np.linspace(0, n_req - 1, n).astype(np.int32))
        ttl = [0.0, float(gaps.min()), float(gaps.max())]
        K.kv_ttl_curves(t, ttl, *out)
        same = np.arange(1, n) // 3 == np.arange(n - 1) // 3
        assert out[0].tolist() == [[int((gaps[same] <= x).sum()) for x in ttl]]
    t.free()
    for at in {0, 1, n_req // 2, n_req - 2, n_req - 1} & set(range(1, n_req)):
        bad = times.clone()
        bad[at] = bad[at - 1] - 0.5
        with pytest.raises(K.KvError, match="request times decreasing"):
            load(n, bad)
    times[-1] = float("nan")
    with pytest.raises(K.KvError, match="request times decreasing"):
        load(n, times)


def test_many_requests_take_the_whole_chip():
    import torch
    from paper_2603_08739_amd import kvcfg as K
    times = torch.arange(50_000_000, device="cuda", dtype=torch.float64)
    load(1000, times).free()
    K.kv_timing_enable(True)
    try:
        K.kv_timing_read(True)
        load(1000, times).free()
        ms = K.kv_timing_read(True)["load_validate"][1]
    finally:
        K.kv_timing_enable(False)
    assert ms < 10, ms  # 0.8 GB read and written; one workgroup alone takes 47 ms
