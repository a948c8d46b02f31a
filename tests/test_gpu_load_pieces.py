"""kv_trace_load where many accesses share partition bits: stretches are cut
into pieces of 8,192 and joined.  Stretch lengths on both sides of one, two
and three pieces, at every alignment the ones before them give; stretches of
one block, of a few and of nearly as many as a linking table holds, and of
more (the load sorts); blocks met in one piece only, in all, and in the first
and last; the block whose hash mixes to zero; one block in every second
access.  Statistics and counts against the oracle (exact)."""
import os

import numpy as np
import pytest

import tracegen as tg
from tests.test_gpu_load_partition import check, unmix

pytestmark = pytest.mark.gpu
PIECE = 8192


def run(O, stretches, bits, label, seed=0):
    """stretches: per value of the top `bits` bits a list of block numbers in order."""
    from paper_2603_08739_amd import host
    rng = np.random.default_rng([seed, bits])
    n = sum(len(s) for s in stretches)
    assert n >> (bits - 1) > 512  # that many partition bits are taken
    which = rng.permutation(np.repeat(np.arange(len(stretches)), [len(s) for s in stretches]))
    h = np.zeros(n, np.uint64)
    for d, s in enumerate(stretches):
        names = {b: unmix((d << (64 - bits)) | int(b)) for b in np.unique(s)} if len(s) else {}
        h[which == d] = [names[b] for b in s]
    t = tg.Trace(label, h, (np.arange(n) // 7).astype(np.uint32), np.zeros(n, np.uint8),
                 np.where(h & np.uint64(1), 1, 4).astype(np.uint8), np.arange((n + 6) // 7, dtype=np.float64) / 4, 1)
    cfgs = tg.from_list([{"cap": (c, 0, 0), "policy": p} for c in (4, 40, 900) for p in range(3)])
    print(f"  case {label}: n={n} stretches={[len(s) for s in stretches]}", flush=True)
    os.environ["KVCFG_TEST_LOAD_BITS"] = str(bits)
    try:
        tr = host.load(t)
    finally:
        os.environ.pop("KVCFG_TEST_LOAD_BITS")
    st = tr.info()
    ids, first, count = np.unique(h, return_index=True, return_counts=True)
    assert (st.n, st.n_distinct, st.max_multiplicity) == (n, len(ids), count.max())
    assert (st.n_w, st.distinct_w) == (t.weight.sum(dtype=np.uint64), t.weight[first].sum(dtype=np.uint64))
    counts, _ = host.evaluate(tr, cfgs, tg.DEFAULT_COST, 1)
    tr.free()
    np.testing.assert_array_equal(counts, O.replay_memo(t, cfgs))


@pytest.mark.parametrize("blocks", [1, 5, 900])
def test_lengths(oracle_mod, blocks):
    rng = np.random.default_rng(blocks)
    for i, lens in enumerate(([PIECE, PIECE + 1, PIECE - 1, 2 * PIECE], [1, 2 * PIECE - 1, 2 * PIECE + 1, 2 * PIECE],
                              [3 * PIECE + 5, 0, 300, 3 * PIECE], [0, 2 * PIECE - 63, 64, 5 * PIECE + 1])):
        run(oracle_mod, [rng.integers(0, blocks, x) for x in lens], 2, f"lengths{i}-{blocks}", i)


def test_blocks_of_parts(oracle_mod):
    """Blocks of the first and last part only, of single parts, in every part;
    the block that mixes to zero (number 0 of the first stretch) among them."""
    a = np.full(6 * PIECE, 7)
    a[[3, 6 * PIECE - 2]] = 0
    a[[10, PIECE * 5 + 1]] = 11
    a[2 * PIECE:2 * PIECE + 300] = np.arange(100, 400)
    a[4 * PIECE + 70:4 * PIECE + 75] = 12
    b = np.zeros(4 * PIECE, int)
    b[::97] = np.arange(len(b[::97])) % 50 + 1
    run(oracle_mod, [a, b], 1, "parts")
    run(oracle_mod, [b, a], 1, "parts-swapped", 1)


@pytest.mark.parametrize("distinct,sorts", [(890, False), (1000, True), (3000, True)])
def test_full_tables(oracle_mod, distinct, sorts):
    """Parts whose tables have room, of a stretch whose table has, or not."""
    from paper_2603_08739_amd import kvcfg as K
    s = np.concatenate([np.r_[x, np.zeros(PIECE, int)] for x in np.array_split(np.arange(distinct), 6)])
    K.kv_timing_enable(True)
    try:
        K.kv_timing_read(True)
        run(oracle_mod, [s, np.arange(800)], 1, f"tables{distinct}")
        assert K.kv_timing_read(True)["load_sort"][0] == (2 if sorts else 1)
    finally:
        K.kv_timing_enable(False)


@pytest.mark.parametrize("n", [8193, 100_000, 700_000])
def test_half_of_one_block(oracle_mod, n):
    from paper_2603_08739_amd import host
    lab = np.where(np.arange(n) % 2, 0, np.random.default_rng(n).integers(1, n // 3, n))
    h = (lab.astype(np.uint64) + np.uint64(1)) * np.uint64(0x9E3779B97F4A7C15)
    t = tg.Trace("half", h, (np.arange(n) // 2).astype(np.uint32), np.zeros(n, np.uint8), np.ones(n, np.uint8),
                 np.arange((n + 1) // 2, dtype=np.float64), 1)
    cfgs = tg.from_list([{"cap": (c, d, 0), "policy": p} for c, d in ((1, 3), (n // 50, n // 5)) for p in range(3)])
    print("  half", n, flush=True)
    tr = host.load(t)
    st = tr.info()
    assert (st.n_distinct, st.max_multiplicity) == (len(np.unique(lab)), np.bincount(lab).max())
    counts, _ = host.evaluate(tr, cfgs, tg.DEFAULT_COST, 1)
    tr.free()
    np.testing.assert_array_equal(counts, oracle_mod.replay_memo(t, cfgs))


@pytest.mark.parametrize("bits,n,u", [(1, 80_000, 40), (1, 300_000, 1200), (4, 300_000, 5000)])
def test_few_partition_bits(oracle_mod, bits, n, u):
    os.environ["KVCFG_TEST_LOAD_BITS"] = str(bits)
    try:
        check(oracle_mod, n, u, groups=2, skew=1.0, seed=bits)
    finally:
        os.environ.pop("KVCFG_TEST_LOAD_BITS")
