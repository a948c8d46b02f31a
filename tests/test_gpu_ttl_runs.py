"""TTL curves: accesses joined into runs of one (request, previous request,
group).  Lengths next to a thread's eight accesses, a wavefront's 512 and a
workgroup's step; requests that re-read one earlier request, several, or a
different one per access; runs cut by new blocks and by group changes; against
the oracle (counts exact, storage to 1e-12: sums of at most 4e4 doubles)."""
import numpy as np
import pytest

import tracegen as tg

pytestmark = pytest.mark.gpu


def labels(kind, n, per):
    i = np.arange(n)
    if kind == "reread":    # every request reads the same blocks again
        return i % per
    if kind == "mixed":     # half re-read, every seventh block new
        return np.where(i % 7 == 3, 10**6 + i, i % per)
    if kind == "strides":   # previous accesses in many earlier requests
        return (i * 37) % (11 * per + 1)
    return np.random.default_rng(n).integers(0, max(2, n // 3), n)


@pytest.mark.parametrize("kind", ["reread", "mixed", "strides", "random"])
@pytest.mark.parametrize("n", [1, 7, 8, 9, 511, 512, 513, 1030, 8191, 8193, 30_011])
def test_runs(oracle_mod, kind, n):
    from paper_2603_08739_amd import host
    for per, groups, weights in ((5, 1, (1,)), (64, 3, (1, 4)), (700, 2, (255, 3))):
        lab = labels(kind, n, per)
        t = tg.from_blocks(lab, weights={int(b): weights[int(b) % len(weights)] for b in np.unique(lab)},
                           groups={int(b): int(b) // 3 % groups for b in np.unique(lab)}, n_groups=groups, per_request=per)
        ttl = [0.0, 0.5, 0.5, 1.0, 2.75, 60.0, 1e6]
        h = host.load(t)
        hits, hitw, store = host.ttl_curves(h, ttl, groups)
        h.free()
        want = oracle_mod.ttl_curves(t, ttl)
        np.testing.assert_array_equal(hits, want[0])
        np.testing.assert_array_equal(hitw, want[1])
        np.testing.assert_allclose(store, want[2], rtol=1e-12, atol=0)
