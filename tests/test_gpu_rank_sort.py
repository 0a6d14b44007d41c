"""MELD_AUTO sorts of 2^12 + 1 .. 2^17 keys (runs and ranks) against the oracle.

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
