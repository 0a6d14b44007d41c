"""MELD_AUTO sorts of 2^12 + 1 .. 2^17 keys and 2^11 + 1 .. 2^16 pairs (runs and ranks) against the oracle.

Bar: bit-exact. Sizes at the edges of a run and of the numbers of runs the kernels are
built for; ties within and across runs, the padding's value, sorted and reversed input;
calls in a row on one context, so that runs of an earlier call would show.
"""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
meld = pytest.importorskip("paper_2107_05681_amd")

SIZES = [(1 << 12) + 1, 5000, 6144, (1 << 13) - 1, 1 << 13, (1 << 13) + 1, 10_000, (1 << 14) - 1, 1 << 14, (1 << 14) + 1, 20_480, (1 << 15) - 3,
         1 << 15, (1 << 15) + 1, 50_001, (1 << 16) - 1, 1 << 16, (1 << 16) + 1, 90_113,
         98_303, 98_304, 98_305, (1 << 17) - 8191, 1 << 17]


def _sort(keys, ctx, sort):
    guard = np.arange(64, dtype=np.uint32)
    buf = torch.from_numpy(np.concatenate([keys, guard]).view(np.int32)).to("cuda:0")
    sort(buf[:len(keys)], variant="auto", ctx=ctx)
    got = buf.cpu().numpy().view(np.uint32)
    assert np.array_equal(got[len(keys):], guard)
    return got[:len(keys)]


def test_sizes_and_orders():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = meld.new_context(0)
    try:
        for n in SIZES[::-1] + SIZES:
            assert meld.sort_plan(n, variant="auto", ctx=ctx)["sorts_by"] == "ranks"
            keys = workloads.keys_u32(n, n)
            ends = keys.copy()
            ends[::3] = 0xFFFFFFFF
            ends[1::5] = 0
            for k in (keys, keys % np.uint32(3), ends, np.sort(keys), np.sort(keys)[::-1],
                      np.zeros(n, np.uint32), np.full(n, 0xFFFFFFFF, np.uint32)):
                k = np.ascontiguousarray(k)
                assert np.array_equal(_sort(k, ctx, meld.sort), oracle.sort_u32(k)), n
            assert np.array_equal(_sort(keys, ctx, meld.merge_sort), oracle.sort_u32(keys)), n
        for n, by in ((1 << 12, "registers"), ((1 << 17) + 1, "radix")):
            assert meld.sort_plan(n, variant="auto", ctx=ctx)["sorts_by"] == by
    finally:
        meld.destroy_context(ctx)


def _sort_pairs(keys, vals, ctx):
    guard = np.arange(64, dtype=np.uint32)
    k, v = (torch.from_numpy(np.concatenate([a, guard]).view(np.int32)).to("cuda:0")
            for a in (keys, vals))
    meld.sort(k[:len(keys)], v[:len(keys)], variant="auto", ctx=ctx)
    k, v = k.cpu().numpy().view(np.uint32), v.cpu().numpy().view(np.uint32)
    assert np.array_equal(k[len(keys):], guard) and np.array_equal(v[len(keys):], guard)
    return k[:len(keys)], v[:len(keys)]


@pytest.mark.parametrize("log", range(1, 17))
def test_pairs(log):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = meld.new_context(0)
    try:
        for n in sorted({max(2, (1 << log) - 1), 1 << log, min(1 << 16, (1 << log) + 1),
                         3 << (log - 1)} - {3 << 15}):
            by = meld.sort_plan(n, pairs=True, variant="auto", ctx=ctx)["sorts_by"]
            assert by == ("registers" if n <= 1 << 11 else "ranks")
            keys, vals = workloads.keys_u32(n, n), workloads.keys_u32(n + 1, n)
            ends, vends = keys % np.uint32(2), vals.copy()
            ends[::3] = vends[::3] = 0xFFFFFFFF
            index = np.arange(n, dtype=np.uint32)
            for k, v in ((keys, vals), (keys % np.uint32(5), index), (ends, vends),
                         (np.sort(keys)[::-1], index[::-1]), (vals & np.uint32(1), keys)):
                k, v = np.ascontiguousarray(k), np.ascontiguousarray(v)
                rk, rv = oracle.sort_pairs_u32(k, v)
                gk, gv = _sort_pairs(k, v, ctx)
                assert np.array_equal(gk, rk) and np.array_equal(gv, rv), n
    finally:
        meld.destroy_context(ctx)
