"""kv_pareto around its tiles of 256 points and wavefronts of 64: sizes next to
their edges, fronts that are everything, almost everything or one row, ties,
segments, bounds and NaN rows, against the all-pairs oracle (exact)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def points(kind, n, rng):
    if kind == "antichain":  # every row on the front
        x = rng.permutation(n).astype(np.float64)
        return np.stack([x, x, np.zeros(n)], axis=1)
    if kind == "chain":      # one row dominates all others
        x = rng.permutation(n).astype(np.float64)
        return np.stack([x, -x, x], axis=1)
    return rng.integers(0, 12 if kind == "ties" else 10_000, (n, 3)).astype(np.float64)


@pytest.mark.parametrize("kind", ["antichain", "chain", "ties", "spread"])
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 255, 256, 257, 511, 513, 2049, 6001])
def test_sizes_at_tile_edges(kind, n, oracle_mod):
    from paper_2603_08739_amd import host, kvcfg as K
    rng = np.random.default_rng([n, len(kind)])
    obj = points(kind, n, rng)
    for seg, bounds in ((None, None), (rng.integers(0, 3, n).astype(np.uint32), None),
                        (None, (n * 0.7, np.nan, np.nan)), (rng.integers(0, 2, n), (np.nan, 3.0, n * 0.9))):
        flags, count = host.pareto(obj, seg, bounds)
        want = oracle_mod.pareto(obj, seg, bounds)
        np.testing.assert_array_equal(flags, want)
        assert count == int(want.sum())
    # NaN rows: flag 0, dominate nothing, reported by the counting call and
    # not by the next one
    bad = obj.copy()
    bad[rng.integers(0, n, 1 + n // 100), rng.integers(0, 3, 1 + n // 100)] = np.nan
    dev = torch.from_numpy(bad).cuda()
    flags = torch.full((n,), 7, dtype=torch.uint8, device="cuda")
    with pytest.raises(K.KvError) as e:
        K.kv_pareto(dev, flags)
    assert e.value.status == K.KV_ERR_INVALID
    ok = ~np.isnan(bad).any(axis=1)
    want = np.zeros(n, np.uint8)
    want[ok] = oracle_mod.pareto(bad[ok])
    np.testing.assert_array_equal(flags.cpu().numpy(), want)
    _, count = host.pareto(obj)
    assert count == int(oracle_mod.pareto(obj).sum())
